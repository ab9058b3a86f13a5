"""The X-update's denominator with more taps and shifts than one filling of the threads takes, in
launches of few and of many frequencies, at widths that are not a multiple of a workgroup's
frequencies.  Through the solve, against float64; the bound is the solve's own (two roundings
per butterfly level and the few products, u = 2^-23)."""
import math

import numpy as np
import pytest
import torch

from paper_2210_04184_amd import nlpr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,q", [(48, 36), (512, 288)])
@pytest.mark.parametrize("r,Sw", [(1, 2), (2, 3), (5, 1), (8, 7)])
def test_denominator_matches_float64(p, q, r, Sw):
    w = 2 * r + 1
    blur = np.random.default_rng(r).uniform(0.0, 1.0, (w, w))
    blur = (blur / blur.sum()).astype(np.float32)
    plan = nlpr.Plan(p, q, 2, 1, 4, blur, np.full((2, 1), 0.5, np.float32), 1, Sw, 1, 1e-3, 1e-2,
                     0.5)
    grid = torch.zeros(p, q, dtype=torch.float64)
    for a in range(-r, r + 1):
        for b in range(-r, r + 1):
            grid[a % p, b % q] += float(blur[a + r, b + r])
    u = torch.arange(p, dtype=torch.float64)[:, None] / p
    v = torch.arange(q, dtype=torch.float64)[None, :] / q
    den = 1.0 + torch.fft.fft2(grid).abs() ** 2
    for t in plan.half_window():
        den += 9 * 2 * (2 - 2 * torch.cos(2 * math.pi * (u * t[0] + v * t[1])))
    C = torch.randn(2, p, q, generator=torch.Generator().manual_seed(r)).cuda()
    X = torch.empty_like(C)
    plan.stage(nlpr.STAGE_XSOLVE, [C, X, plan.alloc_workspace()])
    ref = torch.fft.ifft2(torch.fft.fft2(C.cpu().double()) / den).real
    bound = 2.0 ** -23 * (2 * math.log2(p * q) + 8)
    assert float((X.cpu().double() - ref).norm() / ref.norm()) <= bound
