"""The X-update's passes at the lengths where their stages differ: one stage (8), a last stage of
radix 8, 4, 2 or 3, powers of 3 only, threads of a line in one wave or not, odd band counts,
several images' worth of column blocks that do not divide the width; and the groups of the fused-S
solve.  Against the same solve in float64.

Tolerance: each of the 2 log2(p q) butterfly levels (forward and inverse) and the few products
(twiddles, weights) rounds once, so the relative error in the 2-norm stays below
u (2 log2(p q) + 8) with u = 2^-23."""
import math

import numpy as np
import pytest
import torch

from paper_2210_04184_amd import nlpr

pytestmark = pytest.mark.gpu

SHAPES = [(8, 8, 1), (9, 12, 3), (8, 64, 2), (27, 36, 3), (16, 512, 1), (64, 8, 5), (96, 48, 2),
          (128, 108, 4), (243, 24, 2), (256, 32, 3), (512, 16, 2), (162, 1024, 1),
          (768, 288, 1), (1024, 96, 2), (8, 4096, 1), (4096, 8, 1), (2048, 36, 1)]


def _plan(p, q, L, d, flags=0):
    g = np.exp(-np.arange(-1, 2) ** 2 / 2.0)
    blur = (np.outer(g, g) / np.outer(g, g).sum()).astype(np.float32)
    return blur, nlpr.Plan(p, q, L, 1, d, blur, np.full((L, 1), 1.0 / L, np.float32), 1, 1, 1,
                           1e-3, 1e-2, 0.5, flags=flags)


def _tables(p, q, blur):
    """b^ and 1 + |P| sum |d^|^2 of the 3x3 patch and window."""
    grid = torch.zeros(p, q, dtype=torch.float64)
    for a in range(-1, 2):
        for b in range(-1, 2):
            grid[a % p, b % q] += float(blur[a + 1, b + 1])
    u = torch.arange(p, dtype=torch.float64)[:, None] / p
    v = torch.arange(q, dtype=torch.float64)[None, :] / q
    a = torch.ones(p, q, dtype=torch.float64)
    for t in ((0, 1), (1, -1), (1, 0), (1, 1)):
        a += 9 * 2 * (2 - 2 * torch.cos(2 * math.pi * (u * t[0] + v * t[1])))
    return torch.fft.fft2(grid), a


def _bound(p, q):
    return 2.0 ** -23 * (2 * math.log2(p * q) + 8)


@pytest.mark.parametrize("p,q,L", SHAPES)
def test_solve_matches_float64(p, q, L):
    blur, plan = _plan(p, q, L, 1)
    C = torch.randn(L, p, q, generator=torch.Generator().manual_seed(p + q)).cuda()
    X = torch.empty_like(C)
    plan.stage(nlpr.STAGE_XSOLVE, [C, X, plan.alloc_workspace()])
    bh, a = _tables(p, q, blur)
    ref = torch.fft.ifft2(torch.fft.fft2(C.cpu().double()) / (a + bh.abs() ** 2)).real
    assert float((X.cpu().double() - ref).norm() / ref.norm()) <= _bound(p, q)


@pytest.mark.parametrize("p,q,L,d", [(8, 8, 1, 2), (24, 36, 3, 3), (96, 64, 2, 4), (64, 96, 1, 8),
                                     (256, 36, 2, 2), (48, 48, 2, 6), (512, 32, 1, 8)])
def test_group_solve_matches_float64(p, q, L, d):
    blur, plan = _plan(p, q, L, d, flags=nlpr.FUSED_S)
    C = torch.randn(L, p, q, generator=torch.Generator().manual_seed(p * q)).cuda()
    X = torch.empty_like(C)
    plan.stage(nlpr.STAGE_XSOLVE, [C, X, plan.alloc_workspace()])
    bh, a = _tables(p, q, blur)
    split = lambda F: F.reshape(F.shape[:-2] + (d, p // d, d, q // d))
    ch, a, b = split(torch.fft.fft2(C.cpu().double())), split(a), split(bh)
    t = (b / a * ch).sum(dim=(-4, -2), keepdim=True)
    g = 1.0 / (1e-2 * d * d + (b.abs() ** 2 / a).sum(dim=(-4, -2), keepdim=True))
    ref = torch.fft.ifft2((ch / a - b.conj() / a * g * t).reshape(L, p, q)).real
    assert float((X.cpu().double() - ref).norm() / ref.norm()) <= _bound(p, q)
