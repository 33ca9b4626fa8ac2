"""KS kernels at the edges of their layout: the packed inverse (two columns per
transform) with and without kappa_B, the large three-step transforms (4096
points, float64 from 1024), and zero-extended fields read and written at
their own size (odd widths, one row or column, a field of the whole grid,
strips and phases that the field ends in, rotation blocks that straddle
rows).

Tolerances: a length-N transform of rounding eps is within 5 eps log2 N of
the exact one in norm (three to four rounded operations per butterfly level);
two forward and two inverse levels sets, the multiply and the twiddles give
(4 * 5 log2 N + 20) eps, relative to the 2-norm over the whole grid, which for
kappa is at most that of the shear (|conj(D)| <= 1); a field's corner can be
far below it (kappa of a single pixel is 0).  The max over the map is taken
against 8 times that over the shear's rms.
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


def shears(ny, nx, seed, npt):
    rng = np.random.default_rng(seed)
    return [rng.standard_normal((ny, nx)).astype(npt) for _ in range(2)]


def check(got, ref, shear, n, npt):
    eps = np.finfo(npt).eps
    tol = (20 * math.log2(n) + 20) * eps
    d = got.cpu().numpy().astype(np.float64) - ref
    scale = np.sqrt(sum(np.mean(g.astype(np.float64) ** 2) for g in shear))
    assert np.sqrt(np.mean(d * d)) <= tol * scale
    assert np.max(np.abs(d)) <= 8 * tol * scale


@pytest.mark.parametrize("npt,n", [(np.float32, 16), (np.float32, 32), (np.float32, 64), (np.float32, 512),
                                   (np.float32, 2048), (np.float32, 4096), (np.float64, 16), (np.float64, 512),
                                   (np.float64, 1024), (np.float64, 2048), (np.float64, 4096)])
def test_kappa_e_and_b(ctx, n, npt):
    print("KS n=%d %s" % (n, npt.__name__), flush=True)
    g1, g2 = shears(n, n, 3 + n, npt)
    t1, t2 = (torch.from_numpy(g).cuda() for g in (g1, g2))
    kE, kB = ctx.ks_invert(t1, t2, want_b=True)
    only, _ = ctx.ks_invert(t1, t2)
    rE, rB = O.ks_invert(g1.astype(np.float64), g2.astype(np.float64))
    check(kE, rE, (g1, g2), n, npt)
    check(kB, rB, (g1, g2), n, npt)
    assert torch.equal(only, kE)


FIELDS = [(1, 1, 16), (3, 16, 16), (16, 5, 32), (37, 53, 64), (100, 99, 256), (255, 129, 512), (513, 7, 1024),
          (1000, 1001, 2048), (9, 2047, 2048), (2049, 33, 4096), (130, 4095, 4096)]


@pytest.mark.parametrize("npt", [np.float32, np.float64])
@pytest.mark.parametrize("ny,nx,P", FIELDS)
def test_fields(ctx, ny, nx, P, npt):
    print("KS field %dx%d in %d %s" % (ny, nx, P, npt.__name__), flush=True)
    g1, g2 = shears(ny, nx, ny + nx, npt)
    t1, t2 = (torch.from_numpy(g).cuda() for g in (g1, g2))
    guard = torch.full((ny * nx + 64,), 7.0, dtype=t1.dtype, device="cuda")
    kE = guard[:ny * nx].view(ny, nx)
    ctx.ks_invert_padded(t1, t2, P, kappa_e=kE)
    assert bool((guard[ny * nx:] == 7.0).all())  # nothing written past the field
    both, kB = ctx.ks_invert_padded(t1, t2, P, want_b=True)
    assert torch.equal(both, kE)
    rE, rB = O.ks_invert_padded(g1.astype(np.float64), g2.astype(np.float64), P)
    check(kE, rE, (g1, g2), P, npt)
    check(kB, rB, (g1, g2), P, npt)


@pytest.mark.parametrize("npt", [np.float32, np.float64])
@pytest.mark.parametrize("ny,nx,P,J", [(21, 13, 32, 3), (40, 33, 64, 3), (301, 203, 512, 4), (33, 1025, 2048, 3),
                                       (1025, 30, 2048, 3), (40, 2051, 4096, 3)])
def test_field_noise_rotation(ctx, ny, nx, P, J, npt):
    """sigma of few realisations against the oracle: the phases follow the
    field's flat pixel index through every strip."""
    print("field noise %dx%d in %d %s" % (ny, nx, P, npt.__name__), flush=True)
    g1, g2 = shears(ny, nx, 11 + ny, npt)
    t1, t2 = (torch.from_numpy(g).cuda() for g in (g1, g2))
    R = 3
    sigma, _ = ctx.noise_maps_bc(t1, t2, P, J, amap.BC_MIRROR, R, 29)
    ref = O.noise_sigma_bc(g1.astype(np.float64), g2.astype(np.float64), P, J, 1, R, 29)
    got = sigma.cpu().numpy().astype(np.float64)
    # each realisation's planes carry the KS error plus the hardware sine and
    # cosine's 1.3e-7 (float32); sigma is within sqrt(R / (R - 1)) of that
    eps = np.finfo(npt).eps
    tol = 2 * ((20 * math.log2(P) + 20) * eps + (1.3e-7 if npt == np.float32 else 0.0))
    scale = np.sqrt(np.mean(g1.astype(np.float64) ** 2 + g2.astype(np.float64) ** 2))
    assert np.max(np.abs(got - ref)) <= 8 * tol * scale
