"""Noise statistics merged at the end from per-batch, per-group partials, at
the edges of that rule: one partial, a last batch with fewer realisations than
groups, many capped batches, more partials than the merge takes (merged batch
by batch instead), sub-grid orders in blocks of part of a row and of several
rows; against the oracle.

Tolerance: a realisation's plane is within (20 log2 n + 20) eps of the exact
one relative to the shear's rms (transforms of log2 n rounded levels each way,
the starlet's averages add less), plus 1.3e-7 for the single-precision hardware
sine and cosine; sigma moves by at most sqrt(R / (R - 1)) <= 1.5 times that,
times 8 for the largest pixel; the running update of R values in the element
type adds R eps of sigma, which is at most the shear's rms.
"""
import math

import numpy as np
import pytest
import torch

import oracle as O
import paper_1204_4293_amd as amap

pytestmark = pytest.mark.gpu

CASES = [
    # n, J, R, cap on the batch (0: default), autotune mode
    (16, 2, 2, 0, 0),
    (16, 4, 7, 3, 0),       # last batch of one
    (16, 3, 1100, 2, 0),    # 550 batches: more partials than one merge takes
    (32, 4, 33, 32, 0),     # last batch smaller than the groups
    (64, 5, 20, 8, 2),      # sub-grid final stage
    (256, 6, 9, 4, 2),
    (256, 7, 5, 0, 1),      # tuned
    (512, 8, 3, 2, 1),
]


@pytest.mark.parametrize("npt", [np.float32, np.float64])
@pytest.mark.parametrize("n,J,R,cap,mode", CASES)
def test_sigma_and_snr(n, J, R, cap, mode, npt):
    print("deferred statistics n=%d J=%d R=%d cap=%d mode=%d %s" % (n, J, R, cap, mode, npt.__name__), flush=True)
    ctx = amap.Context(0)
    ctx.set_autotune(mode)
    ctx.set_noise_batch(cap)
    rng = np.random.default_rng(n + R)
    g1, g2 = (rng.standard_normal((n, n)).astype(npt) for _ in range(2))
    t1, t2 = (torch.from_numpy(g).cuda() for g in (g1, g2))
    kappa, _ = ctx.ks_invert(t1, t2)
    planes = ctx.starlet_forward(kappa, J)
    for again in range(2):  # the second pass finds the first one's partials in the workspace
        sigma, snr = ctx.noise_maps(t1, t2, J, R, 71, planes_signal=planes)
    ref = O.noise_sigma(g1.astype(np.float64), g2.astype(np.float64), J, R, 71)
    got = sigma.cpu().numpy().astype(np.float64)
    eps = np.finfo(npt).eps
    rms = np.sqrt(np.mean(g1.astype(np.float64) ** 2 + g2.astype(np.float64) ** 2))
    w_tol = (20 * math.log2(n) + 20) * eps + (1.3e-7 if npt == np.float32 else 0.0)
    tol = (8 * 1.5 * w_tol + R * eps) * rms
    assert np.max(np.abs(got - ref)) <= tol
    w = planes[:-1].cpu().numpy()
    s = sigma.cpu().numpy()
    expect = np.where(s > 0, w / np.where(s > 0, s, 1), 0).astype(npt)
    assert np.allclose(snr.cpu().numpy(), expect, rtol=4 * eps, atol=0)
    ctx.close()
