"""A map in a batch plan against the same map alone, bit for bit, on both sides
of every batch size at which a launch changes its shape: 128^2 and 256^2 row
passes around 4096 row pairs, 2048^2 forward strips (float32), and the widths
of the column strips.  A launch may spread its work differently for a larger
batch; the arithmetic of each map may not depend on it.
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


def shear(n, dtype, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return [(0.07 * torch.randn((n, n), generator=g, device="cuda", dtype=torch.float64)).to(dtype) for _ in range(2)]


@pytest.mark.parametrize("dtype,n,count", [
    (torch.float32, 128, 64), (torch.float32, 128, 65), (torch.float64, 128, 65),
    (torch.float32, 256, 32), (torch.float32, 256, 33), (torch.float64, 256, 33),
    (torch.float32, 512, 3), (torch.float32, 512, 40), (torch.float64, 512, 9),
    (torch.float32, 1024, 2), (torch.float32, 1024, 9), (torch.float64, 1024, 3),
    (torch.float32, 2048, 2), (torch.float32, 2048, 3), (torch.float32, 2048, 4), (torch.float32, 2048, 5),
    (torch.float64, 2048, 2),
])
def test_grouped_map_is_the_map_alone(ctx, dtype, n, count):
    J = 4
    jobs = []
    for i in range(count):
        g1, g2 = shear(n, dtype, 100 * n + i)
        jobs.append({"g1": g1, "g2": g2, "kappa_e": torch.full((n, n), float("nan"), dtype=dtype, device="cuda"),
                     "planes": torch.full((J, n, n), float("nan"), dtype=dtype, device="cuda")})
    plan = amap.BatchPlan(ctx, jobs)
    plan.run()
    ctx.sync()
    for i in sorted({0, 1, count // 2, count - 1}):
        kappa, _ = ctx.ks_invert(jobs[i]["g1"], jobs[i]["g2"])
        planes = ctx.starlet_forward(kappa, J)
        assert torch.equal(jobs[i]["kappa_e"], kappa), i
        assert torch.equal(jobs[i]["planes"], planes), i
    plan.close()
