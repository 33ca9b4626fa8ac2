"""Peak and moment kernels where their blocks stride over a plane more than
once, against the oracle on identical planes: counts of fields of more than 256
blocks (2^20 floats or 2^19 doubles), with odd pixel counts so that planes start
off a 16-byte boundary; histograms of more blocks than a plane gets; moments
past the first unrolled pass.
"""
import numpy as np
import pytest
import torch

import oracle as O
import paper_1204_4293_amd as amap

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    c = amap.Context(0)
    yield c
    c.close()


def planes_of(count, ny, nx, dtype, seed):
    rng = np.random.default_rng(seed)
    a = rng.standard_normal((count, ny, nx))
    a[0] = np.round(4.0 * a[0]) / 4.0  # many ties
    return a.astype(dtype)


@pytest.mark.parametrize("dtype,ny,nx", [(np.float64, 1021, 1023), (np.float32, 1101, 1003)])
@pytest.mark.parametrize("mode", [amap.BC_PERIODIC, amap.BC_MIRROR, amap.BC_ZERO])
def test_counts_of_large_fields(ctx, dtype, ny, nx, mode):
    a = planes_of(2, ny, nx, dtype, ny)
    mask = (np.random.default_rng(nx).random((ny, nx)) > 0.02).astype(np.uint8)
    t, m = torch.from_numpy(a).cuda(), torch.from_numpy(mask).cuda()
    for thr in (-10.0, 2.0):
        got = ctx.count_peaks_bc(t, thr, mode).cpu().tolist()
        assert got == [O.count_peaks_bc(p.astype(np.float64), thr, mode) for p in a]
        got = ctx.count_peaks_masked(t, m, thr, mode).cpu().tolist()
        assert got == [O.count_peaks_masked(p.astype(np.float64), thr, mode, mask) for p in a]


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("sign", [1, -1])
def test_histogram_of_many_planes(ctx, dtype, sign):
    a = planes_of(4, 2048, 2048, dtype, 3)
    got = ctx.peak_histogram(torch.from_numpy(a).cuda(), -2.0, 6.0, 40, sign=sign).cpu().numpy()
    assert np.array_equal(got, O.peak_histogram_planes(a.astype(np.float64), -2.0, 6.0, 40, sign))


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_moments_of_large_planes(ctx, dtype):
    """Each sum of n^2 doubles is within n^2 eps of its sum of absolute values."""
    n = 2048
    a = planes_of(2, n, n, dtype, 8) + dtype(0.25)
    got = ctx.plane_moments(torch.from_numpy(a).cuda()).cpu().numpy()
    ref = O.plane_moments_stack(a.astype(np.float64))
    for p in range(2):
        d = np.abs(a[p].astype(np.float64) - ref[p, 0])
        for k in range(4):
            size = np.mean(np.abs(a[p].astype(np.float64))) if k == 0 else np.mean(d ** (k + 1))
            assert abs(got[p, k] - ref[p, k]) <= n * n * 2.3e-16 * size
