"""Rounding error of the KS inversion against long double transforms.

The rms error of a transform grows like u sqrt(log2 n) (u the unit roundoff);
the factor depends on how the twiddles are made.  A model of the passes on the
CPU gives 1.19 where every twiddle of a radix-4 pass is a rounded table value
(double from 1024 points), 1.5 to 1.7 where they are products of two (float,
and double below), and 1.6 to 1.8 with products of three.  The bounds lie
between the kind that runs and the next.
"""
import numpy as np
import pytest
import torch

import paper_1204_4293_amd as amap

pytestmark = pytest.mark.gpu


def exact(g1, g2):
    n = g1.shape[0]
    m = np.arange(n)
    m = np.where(m < n // 2, m, m - n).astype(np.longdouble)
    m1, m2 = m[None, :], m[:, None]
    den = m1 * m1 + m2 * m2
    den[0, 0] = 1
    cross = 2 * m1 * m2
    cross[n // 2, :] = 0
    cross[:, n // 2] = 0
    conj_d = ((m1 * m1 - m2 * m2) / den - 1j * (cross / den)).astype(np.clongdouble)
    g = g1.astype(np.clongdouble) + np.clongdouble(1j) * g2.astype(np.clongdouble)
    return np.fft.ifft2(np.fft.fft2(g) * conj_d).real


@pytest.mark.parametrize("dtype,n,factor", [
    (torch.float32, 128, 1.72), (torch.float32, 512, 1.72), (torch.float32, 1024, 1.72), (torch.float32, 2048, 1.72),
    (torch.float64, 512, 1.6), (torch.float64, 1024, 1.3), (torch.float64, 2048, 1.3),
])
def test_rms_error(dtype, n, factor):
    ctx = amap.Context(0)
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    g1, g2 = ((0.07 * torch.randn((n, n), generator=g, device="cuda", dtype=torch.float64)).to(dtype) for _ in range(2))
    kappa, _ = ctx.ks_invert(g1, g2)
    ctx.sync()
    want = exact(g1.cpu().numpy(), g2.cpu().numpy())
    err = kappa.cpu().numpy().astype(np.longdouble) - want
    rel = float(np.sqrt(np.mean(err * err) / np.mean(want * want)))
    u = float(torch.finfo(dtype).eps) / 2
    assert rel <= factor * u * np.sqrt(np.log2(n)), rel / (u * np.sqrt(np.log2(n)))
    ctx.close()
