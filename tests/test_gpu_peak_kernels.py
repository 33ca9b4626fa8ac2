"""Peak kernels at the edges of their layout, bit-exact against the oracle on
identical planes: fields whose planes start off a 16-byte boundary (odd pixel
counts), shorter than one vector, and over several blocks; histograms of maps
of one strip and of several blocks; ties, NaN, infinities, a threshold that
every pixel passes."""
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


def planes_of(count, ny, nx, dtype, seed):
    rng = np.random.default_rng(seed)
    a = np.round(rng.standard_normal((count, ny, nx)) * 4.0) / 4.0  # many ties
    a[0].flat[ny * nx // 2] = np.nan
    a[0].flat[0] = np.inf
    a[-1].flat[-1] = 9.0
    if count > 1:
        a[1] += rng.standard_normal((ny, nx)) * 1e-3  # no ties
    return a.astype(dtype)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("ny,nx", [(2, 2), (3, 5), (2, 9), (17, 31), (64, 64), (101, 203)])
def test_count_peaks_bc_edges(ctx, ny, nx, dtype):
    a = planes_of(3, ny, nx, dtype, 5 + ny)
    rng = np.random.default_rng(ny * nx)
    mask = (rng.random((ny, nx)) > 0.05).astype(np.uint8)
    t, m = torch.from_numpy(a).cuda(), torch.from_numpy(mask).cuda()
    for mode in (amap.BC_PERIODIC, amap.BC_MIRROR, amap.BC_ZERO):
        for thr in (-1e30, 1.0):
            print("count_peaks_bc %dx%d mode %d thr %g" % (ny, nx, mode, thr), flush=True)
            got = ctx.count_peaks_bc(t, thr, mode).cpu().tolist()
            assert got == [O.count_peaks_bc(p.astype(np.float64), thr, mode) for p in a]
            got = ctx.count_peaks_masked(t, m, thr, mode).cpu().tolist()
            assert got == [O.count_peaks_masked(p.astype(np.float64), thr, mode, mask) for p in a]


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n", [16, 32, 128, 512])
def test_peak_histogram_edges(ctx, n, dtype):
    a = planes_of(2, n, n, dtype, 9 + n)
    t = torch.from_numpy(a).cuda()
    for sign in (1, -1):
        for lo, hi, nbins in ((-2.0, 6.0, 40), (0.0, 1.0, 1), (-5.0, 5.0, 3000)):
            print("peak_histogram n=%d sign %d bins %d" % (n, sign, nbins), flush=True)
            got = ctx.peak_histogram(t, lo, hi, nbins, sign=sign).cpu().numpy()
            assert np.array_equal(got, O.peak_histogram_planes(a.astype(np.float64), lo, hi, nbins, sign))


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n", [16, 32, 64, 128, 1024])
def test_plane_moments_blocks(ctx, n, dtype):
    """One block, a block with a remainder of its unrolled loop, many blocks.
    Each sum of n^2 doubles is within n^2 eps of its sum of absolute values."""
    rng = np.random.default_rng(n)
    a = (rng.standard_normal((2, n, n)) + 0.25).astype(dtype)
    got = ctx.plane_moments(torch.from_numpy(a).cuda()).cpu().numpy()
    ref = O.plane_moments_stack(a.astype(np.float64))
    for p in range(2):
        d = np.abs(a[p].astype(np.float64) - ref[p, 0])
        for k in range(4):
            size = np.mean(np.abs(a[p].astype(np.float64))) if k == 0 else np.mean(d ** (k + 1))
            assert abs(got[p, k] - ref[p, k]) <= n * n * 2.3e-16 * size
