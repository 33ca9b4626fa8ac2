"""Bounded noise statistics kept in the tiles, at the edges of their layout:
fields narrower than a tile, one column over, fewer rows than a residue class
holds, dilations in every column-chunk class and beyond the tiles (row and
column passes), several batches, under every edge rule, against the oracle.

Tolerance: a realisation's plane is within (20 log2 P + 20) eps of the exact
one relative to the shear's rms, plus 1.3e-7 for the single-precision hardware
sine and cosine; sigma moves by at most sqrt(R / (R - 1)) <= 1.5 times that,
times 8 for the largest pixel.
"""
import math

import numpy as np
import pytest
import torch

import oracle as O
import paper_1204_4293_amd as amap

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = amap.Context(0)
    yield c
    c.close()


CASES = [
    # ny, nx, P, J, R
    (2, 2, 16, 2, 2),
    (5, 63, 64, 4, 3),
    (70, 65, 128, 6, 4),     # one column over a tile, d = 16
    (33, 200, 256, 7, 3),    # d = 32
    (129, 140, 256, 9, 2),   # d = 128: the last tiled dilation in float, rows and columns in double
    (150, 131, 256, 10, 2),  # d = 256: beyond the tiles in both
    (40, 50, 64, 5, 37),     # more realisations than one batch
]


@pytest.mark.parametrize("npt", [np.float32, np.float64])
@pytest.mark.parametrize("ny,nx,P,J,R", CASES)
def test_sigma_and_snr(ctx, ny, nx, P, J, R, npt):
    rng = np.random.default_rng(ny * nx)
    g1, g2 = (rng.standard_normal((ny, nx)).astype(npt) for _ in range(2))
    t1, t2 = (torch.from_numpy(g).cuda() for g in (g1, g2))
    eps = np.finfo(npt).eps
    rms = np.sqrt(np.mean(g1.astype(np.float64) ** 2 + g2.astype(np.float64) ** 2))
    tol = 12 * ((20 * math.log2(P) + 20) * eps + (1.3e-7 if npt == np.float32 else 0.0)) * rms
    kappa, _ = ctx.ks_invert_padded(t1, t2, P)
    for mode in (0, 1, 2):
        print("bounded statistics %dx%d J=%d R=%d mode=%d %s" % (ny, nx, J, R, mode, npt.__name__), flush=True)
        planes = ctx.starlet_forward_bc(kappa, J, mode)
        sigma, snr = ctx.noise_maps_bc(t1, t2, P, J, mode, R, 5, planes_signal=planes)
        ref = O.noise_sigma_bc(g1.astype(np.float64), g2.astype(np.float64), P, J, mode, R, 5)
        s = sigma.cpu().numpy()
        assert np.max(np.abs(s.astype(np.float64) - ref)) <= tol
        w = planes[:-1].cpu().numpy().astype(np.float64)
        s64 = s.astype(np.float64)
        expect = np.where(s64 > 0, w / np.where(s64 > 0, s64, 1), 0)
        assert np.allclose(snr.cpu().numpy(), expect, rtol=8 * eps, atol=0)
