"""Bounded noise statistics on both sides of the size from which a tile keeps
its pixels' statistics over the realisations (600 tiles of 64 x 16 pixels),
with dilations beyond the tiles and several batches, against the oracle.
Fields below it are those of test_gpu_bounded_stats.py; the same tolerance."""
import math

import numpy as np
import pytest
import torch

import oracle as O
import paper_1204_4293_amd as amap

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ny,nx,P,J,R,mode,npt", [
    (950, 641, 1024, 10, 3, 1, np.float32),   # 660 tiles, dilation 256
    (950, 641, 1024, 9, 3, 2, np.float64),
    (944, 640, 1024, 4, 3, 0, np.float32),    # 590: stored details, nothing left over
    (945, 640, 1024, 4, 3, 1, np.float64),    # 600, one row in the last tiles
    (950, 641, 2048, 3, 15, 1, np.float64),   # two batches
])
def test_sigma_and_snr(ny, nx, P, J, R, mode, npt):
    print("bounded statistics %dx%d P=%d J=%d R=%d mode=%d %s" % (ny, nx, P, J, R, mode, npt.__name__), flush=True)
    ctx = amap.Context(0)
    rng = np.random.default_rng(ny * nx)
    g1, g2 = (rng.standard_normal((ny, nx)).astype(npt) for _ in range(2))
    t1, t2 = (torch.from_numpy(g).cuda() for g in (g1, g2))
    eps = np.finfo(npt).eps
    rms = np.sqrt(np.mean(g1.astype(np.float64) ** 2 + g2.astype(np.float64) ** 2))
    tol = 12 * ((20 * math.log2(P) + 20) * eps + (1.3e-7 if npt == np.float32 else 0.0)) * rms
    kappa, _ = ctx.ks_invert_padded(t1, t2, P)
    planes = ctx.starlet_forward_bc(kappa, J, mode)
    sigma, snr = ctx.noise_maps_bc(t1, t2, P, J, mode, R, 5, planes_signal=planes)
    ref = O.noise_sigma_bc(g1.astype(np.float64), g2.astype(np.float64), P, J, mode, R, 5)
    s = sigma.cpu().numpy()
    assert np.max(np.abs(s.astype(np.float64) - ref)) <= tol
    w = planes[:-1].cpu().numpy().astype(np.float64)
    s64 = s.astype(np.float64)
    expect = np.where(s64 > 0, w / np.where(s64 > 0, s64, 1), 0)
    assert np.allclose(snr.cpu().numpy(), expect, rtol=8 * eps, atol=0)
    ctx.close()
