"""Tile schedules of noise statistics that are merged at the end and batch by
batch: each is tuned for itself, whichever ran first, and a loaded schedule
serves both.
"""
import pytest
import torch

import paper_1204_4293_amd as amap

pytestmark = pytest.mark.gpu

N, J, CAP = 16, 3, 2
FEW, MANY = 6, 1100  # batches of 2: 3, merged at the end; 550, too many partials for that


def run(ctx, R):
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    g1, g2 = (torch.randn((N, N), generator=g, device="cuda") for _ in range(2))
    sigma, _ = ctx.noise_maps(g1, g2, J, R, 5, want_snr=False)
    ctx.sync()
    return sigma


def context():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    c = amap.Context(0)
    c.set_noise_batch(CAP)
    return c


def modes(ctx):
    return sorted(p["noise"] for p in ctx.plans())


@pytest.mark.parametrize("first,second", [(FEW, MANY), (MANY, FEW)])
def test_each_mode_has_its_own_schedule(first, second):
    ctx = context()
    run(ctx, first)
    run(ctx, second)
    assert 1 in modes(ctx) and 2 in modes(ctx)
    ctx.close()


def test_loaded_schedule_serves_both_modes():
    ctx, other = context(), context()
    run(ctx, FEW)
    plan = [p for p in ctx.plans() if p["noise"] == 1]
    assert len(plan) == 1
    other.plans_load(plan)
    for R in (FEW, MANY):
        run(other, R)
        assert other.plans() == plan
    # one of its own for batch by batch goes before it, and survives a round trip
    own = dict(plan[0], noise=2)
    other.plans_load([own])
    assert other.plans() == plan + [own]
    with pytest.raises(amap.AmapError):
        other.plans_load([dict(own, noise=3)])
    with pytest.raises(amap.AmapError):
        other.plans_load([dict(own, mode=2)])
    ctx.close()
    other.close()
