"""A NaN or an infinity in the shear reaches exactly the outputs whose disc of
offsets |d| <= cut holds it: the direct aperture-mass sum walks the taps of a
row in groups of four, and the taps of a group that lie outside the disc may
not take part, not even with a zero weight.
"""
import pytest
import torch

import paper_1204_4293_amd as amap

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    c = amap.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("n,cut", [(16, 2.0), (64, 9.4), (256, 6.0), (256, 17.0), (512, 4.0), (512, 33.3), (1024, 1.0)])
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_only_discs_that_hold_it(ctx, n, cut, dtype, value):
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    g1, g2 = (torch.randn((n, n), generator=g, device="cuda", dtype=torch.float64).to(dtype) for _ in range(2))
    y, x = n // 2 + 1, n - 2  # the disc wraps round the edge
    for a in (g1, g2):
        a[y, x] = 0.0
    clean = ctx.map_direct(g1, g2, cut / 2.0, amap.FILTER_STARLET, 0.0, cut)
    for a in (g1, g2):
        a[y, x] = value
    out = ctx.map_direct(g1, g2, cut / 2.0, amap.FILTER_STARLET, 0.0, cut)
    i = torch.arange(n, device="cuda")
    dy, dx = ((i - y + n // 2) % n - n // 2)[:, None], ((i - x + n // 2) % n - n // 2)[None, :]
    inside = dy * dy + dx * dx <= cut * cut
    assert torch.equal(out[~inside], clean[~inside])
    assert not torch.isfinite(out[inside]).any()
