"""Row passes of 128 and 256 points: few rows in three steps, many in four
(from more than 4096 pairs of rows), with and without kappa_B, whole maps and
fields, against the oracle.  Tolerances as in test_gpu_ks_layouts.py."""
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


def scale_of(g):
    return np.sqrt(sum(np.mean(x.astype(np.float64) ** 2) for x in g))


@pytest.mark.parametrize("npt", [np.float32, np.float64])
@pytest.mark.parametrize("ny,nx,P", [(128, 128, 128), (256, 256, 256), (77, 100, 128), (1, 128, 128), (130, 3, 256)])
def test_one_map(ctx, ny, nx, P, npt):
    print("KS rows %dx%d in %d %s" % (ny, nx, P, npt.__name__), flush=True)
    g = shears(ny, nx, ny + 3 * nx, npt)
    t1, t2 = (torch.from_numpy(x).cuda() for x in g)
    call = ctx.ks_invert if ny == P and nx == P else lambda a, b, **k: ctx.ks_invert_padded(a, b, P, **k)
    only, _ = call(t1, t2)
    kE, kB = call(t1, t2, want_b=True)
    assert torch.equal(only, kE)
    ref = O.ks_invert_padded(g[0].astype(np.float64), g[1].astype(np.float64), P)
    tol = (20 * math.log2(P) + 20) * np.finfo(npt).eps * scale_of(g)
    for got, r in ((kE, ref[0]), (kB, ref[1])):
        d = got.cpu().numpy().astype(np.float64) - r
        assert np.sqrt(np.mean(d * d)) <= tol * math.sqrt(P * P / (ny * nx))
        assert np.max(np.abs(d)) <= 8 * tol


@pytest.mark.parametrize("npt", [np.float32, np.float64])
@pytest.mark.parametrize("n,R", [(128, 64), (128, 65), (256, 32), (256, 33)])  # 4096 pairs of rows, one map more
def test_batches(ctx, n, R, npt):
    print("noise rows n=%d R=%d %s" % (n, R, npt.__name__), flush=True)
    g = shears(n, n, n + R, npt)
    t1, t2 = (torch.from_numpy(x).cuda() for x in g)
    sigma, _ = ctx.noise_maps(t1, t2, 3, R, 17)
    ref = O.noise_sigma_bc(g[0].astype(np.float64), g[1].astype(np.float64), n, 3, 0, R, 17)
    tol = 2 * ((20 * math.log2(n) + 20) * np.finfo(npt).eps + (1.3e-7 if npt == np.float32 else 0.0))
    assert np.max(np.abs(sigma.cpu().numpy().astype(np.float64) - ref)) <= 8 * tol * scale_of(g)
