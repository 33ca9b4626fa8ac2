"""Final write-mode stages on whole sub-grids (strips of adjacent ones): explicit
schedules against the analytic planner's tiles, whose values they reproduce
bit for bit (every B3 pass adds the same terms in the same order and scales by
powers of two), for every strip shape, one to three scales, single maps and
grouped ones; and the schedules that must be refused."""
import pytest
import torch

import synth as S
import paper_1204_4293_amd as amap

pytestmark = pytest.mark.gpu

# n, J, first scale of the final stage, element type
CASES = [
    (512, 6, 5, torch.float32),     # m = 32, 16 columns: one strip per row residue
    (512, 7, 5, torch.float32),     # two scales
    (1024, 8, 5, torch.float32),    # m = 64, three scales
    (2048, 9, 6, torch.float32),
    (2048, 8, 7, torch.float32),
    (256, 6, 4, torch.float64),     # m = 32, 8 columns
    (512, 8, 5, torch.float64),     # three scales
    (512, 7, 4, torch.float64),     # m = 64, 4 columns
    (2048, 9, 7, torch.float64),
]


def head(n, j0, dtype):
    """Stages of scales 1 .. j0-1, as a context tunes them."""
    ctx = amap.Context(0)
    ctx.starlet_forward(torch.zeros((n, n), dtype=dtype, device="cuda"), j0)
    got = [p["stages"] for p in ctx.plans() if p["noise"] == 0 and p["J"] == j0]
    ctx.close()
    return [s for s in got[0] if s[5] == 0] if all(s[5] == 0 for s in got[0]) else None


@pytest.mark.parametrize("n,J,j0,dtype", CASES)
def test_strips_match_tiles(n, J, j0, dtype):
    print("strips n=%d J=%d from %d %s" % (n, J, j0, dtype), flush=True)
    m = n >> (j0 - 1)
    stages = head(n, j0, dtype)
    if stages is None:  # the head itself was tuned to end in a strip: plain single-scale tiles
        stages = [[j, 1, 128, 16, 1, 0] for j in range(1, j0)]
    stages = stages + [[j0, J - j0, m, m, 1, 1]]
    elem = 4 if dtype == torch.float32 else 8
    logn = n.bit_length() - 1
    ctx = amap.Context(0)
    ctx.plans_load([{"mode": 1, "elem": elem, "logn": logn, "J": J, "noise": 0, "batch": b, "stages": stages}
                    for b in (1, 3)])
    plain = amap.Context(0)
    plain.set_autotune(False)
    kappa = [torch.tensor(S.grf_kappa(n, 5 + k), dtype=dtype, device="cuda") for k in range(3)]
    ref = [plain.starlet_forward(k, J) for k in kappa]
    assert torch.equal(ctx.starlet_forward(kappa[0], J), ref[0])
    # grouped: the same planes from a batch plan of the maps' shears
    jobs = []
    for k in range(3):
        _, g1, g2 = S.shear_map(n, 5 + k)
        jobs.append({"g1": torch.tensor(g1, dtype=dtype, device="cuda"),
                     "g2": torch.tensor(g2, dtype=dtype, device="cuda"),
                     "kappa_e": torch.empty((n, n), dtype=dtype, device="cuda"),
                     "planes": torch.empty((J, n, n), dtype=dtype, device="cuda")})
    plan = amap.BatchPlan(ctx, jobs)
    plan.run()
    torch.cuda.synchronize()
    for j in jobs:
        assert torch.equal(j["planes"], plain.starlet_forward(j["kappa_e"], J))
    plan.close()
    ctx.close()
    plain.close()


@pytest.mark.parametrize("stages", [
    [[1, 1, 128, 16, 1, 0], [2, 5, 256, 256, 1, 1]],                       # sub-grid side without a strip
    [[1, 1, 128, 16, 1, 0], [2, 1, 128, 16, 1, 0], [3, 1, 128, 16, 1, 0], [4, 1, 128, 16, 1, 0],
     [5, 2, 32, 32, 2, 1]],                                                # two maps per pass
    [[1, 1, 128, 16, 1, 0], [2, 1, 128, 16, 1, 0], [3, 1, 128, 16, 1, 0], [4, 1, 128, 16, 1, 0],
     [5, 1, 32, 32, 1, 1], [6, 1, 128, 16, 1, 0]],                         # not the last stage
])
def test_refused_schedules(stages):
    ctx = amap.Context(0)
    with pytest.raises(amap.AmapError):
        ctx.plans_load([{"mode": 1, "elem": 4, "logn": 9, "J": 7, "noise": 0, "batch": 1, "stages": stages}])
    ctx.close()
