"""Write-mode tile stages with more halo than pixels (2.6 to 5 LDS elements per
output pixel), which the tuner offers for signals: explicit schedules against
the analytic planner's tiles, whose values they reproduce bit for bit (every
B3 pass adds the same terms in the same order); tiles beyond the limit, and
the same tiles for noise stages, stay refused."""
import pytest
import torch

import synth as S
import paper_1204_4293_amd as amap

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,J,dtype,stages", [
    (64, 4, torch.float64, [[1, 2, 16, 8, 1, 0], [3, 1, 16, 16, 1, 0]]),
    (64, 4, torch.float32, [[1, 3, 32, 32, 1, 0]]),
    (256, 5, torch.float64, [[1, 3, 32, 32, 1, 0], [4, 1, 32, 8, 1, 0]]),
    (256, 6, torch.float32, [[1, 2, 16, 16, 1, 0], [3, 2, 32, 16, 1, 0], [5, 1, 64, 4, 1, 0]]),
    (512, 6, torch.float32, [[1, 3, 32, 32, 1, 0], [4, 2, 64, 16, 1, 0]]),
])
def test_small_tiles_match(n, J, dtype, stages):
    print("tiles n=%d J=%d %s %s" % (n, J, dtype, stages), flush=True)
    ctx = amap.Context(0)
    ctx.plans_load([{"mode": 1, "elem": 4 if dtype == torch.float32 else 8, "logn": n.bit_length() - 1,
                     "J": J, "noise": 0, "batch": 1, "stages": stages}])
    plain = amap.Context(0)
    plain.set_autotune(False)
    kappa = torch.tensor(S.grf_kappa(n, 7), dtype=dtype, device="cuda")
    assert torch.equal(ctx.starlet_forward(kappa, J), plain.starlet_forward(kappa, J))
    ctx.close()
    plain.close()


@pytest.mark.parametrize("noise,stages", [
    (0, [[1, 3, 16, 8, 1, 0]]),   # 48 x 36 loaded for 16 x 8
    (1, [[1, 3, 32, 32, 1, 0]]),  # a noise stage keeps the smaller limit
])
def test_refused(noise, stages):
    ctx = amap.Context(0)
    with pytest.raises(amap.AmapError):
        ctx.plans_load([{"mode": 1, "elem": 4, "logn": 8, "J": 4, "noise": noise, "batch": 1 + 7 * noise,
                         "stages": stages}])
    ctx.close()
