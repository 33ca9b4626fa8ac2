"""The direct aperture-mass kernel at the edges of its layout: several rows in
one wavefront (sides under 256), one segment per row and several, the largest
cut a side takes, cuts whose padded width changes, and every split of the row
offsets, against the oracle's brute-force sum.

Tolerance: a sum of N products in any order is within N eps sum |w| |g| of the
exact one (first order), with one more rounding each for the weight and for
the sum of two rows: (N + 2) eps sum |w| max |g|, N the taps inside the cut.
"""
import numpy as np
import pytest
import torch

import oracle as O

pytestmark = pytest.mark.gpu

CASES = [
    # n, theta, filter, fparam, cut
    (16, 3.0, O.FILTER_STARLET, 0.0, 7.0),      # 16 rows in a wavefront, largest cut
    (16, 0.4, O.FILTER_STARLET, 0.0, 0.0),      # cut 0.8: no offset inside
    (32, 2.0, O.FILTER_S98, 1.0, 1.0),
    (64, 4.0, O.FILTER_JBJ04, 0.5, 20.3),
    (128, 9.0, O.FILTER_STARLET, 0.0, 63.0),
    (256, 2.5, O.FILTER_STARLET, 0.0, 0.0),     # one segment per row
    (512, 2.0, O.FILTER_STARLET, 0.0, 4.0),
    (512, 3.0, O.FILTER_S98, 2.0, 3.0),         # fewer row offsets than wavefronts
    (1024, 1.3, O.FILTER_STARLET, 0.0, 2.6),    # two segments per row
]


@pytest.fixture(scope="module")
def ctx():
    import paper_1204_4293_amd as amap
    c = amap.Context(0)
    yield c
    c.close()


def sample_points(n, rng):
    edge = [(0, 0), (0, n - 1), (n - 1, 0), (n - 1, n - 1), (n // 2, n // 2 - 1), (n // 2 - 1, n // 2)]
    return edge + [(int(rng.integers(0, n)), int(rng.integers(0, n))) for _ in range(120)]


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("n,theta,filt,fparam,cut", CASES)
def test_direct_rows(ctx, n, theta, filt, fparam, cut, dtype):
    rng = np.random.default_rng(77 + n)
    npt = np.float32 if dtype == torch.float32 else np.float64
    g1, g2 = (rng.standard_normal((n, n)).astype(npt) for _ in range(2))
    print("direct rows n=%d theta=%g cut=%g %s" % (n, theta, cut, dtype), flush=True)
    got = ctx.map_direct(torch.from_numpy(g1).cuda(), torch.from_numpy(g2).cuda(), theta, filt, fparam, cut)
    got = got.cpu().numpy().astype(np.float64)
    pts = sample_points(n, rng)
    ref = O.map_direct_at(g1.astype(np.float64), g2.astype(np.float64), theta, pts, filt, fparam, cut)
    # sum |w| over the taps: the response to a field of unit shear along each tap's phase, bounded by sum |Q|
    c = cut if cut > 0 else {O.FILTER_STARLET: 2.0, O.FILTER_S98: 1.0, O.FILTER_JBJ04: 5.0}[filt] * theta
    R = int(c)
    dy, dx = np.mgrid[-R:R + 1, -R:R + 1]
    r = np.sqrt(dx * dx + dy * dy)
    inside = (r > 0) & (r * r <= c * c)
    taps = int(inside.sum())
    q = {O.FILTER_STARLET: lambda v: O.starlet_Q(v / theta) / theta ** 2,
         O.FILTER_S98: lambda v: O.s98_Q(v, theta, fparam),
         O.FILTER_JBJ04: lambda v: O.jbj04_Q(v, theta, fparam)}[filt]
    sum_w = 2.0 * sum(abs(float(q(v))) for v in r[inside])
    tol = (2 * taps + 2) * np.finfo(npt).eps * sum_w * max(np.abs(g1).max(), np.abs(g2).max())
    for (y, x), v in zip(pts, ref):
        assert abs(got[y, x] - v) <= tol, (y, x, got[y, x], v, tol)
