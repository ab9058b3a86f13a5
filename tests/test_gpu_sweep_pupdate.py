"""The P-update in the sweep's launch: a plan with stage timing runs the two as kernels of their
own, the plain one in one launch, with the same operations in the same order, so X, the dual
state and both Lambda are equal bit for bit.  The shapes have P-update workgroups that end past
the last pixel, sweep tiles that need less LDS than the P-update's exchange of shares, band
shares that are empty or full, every patch radius that shares the launch, and a dual state under
each cache policy; in the last two the plan without timing would otherwise use a second stream."""
import numpy as np
import pytest
import torch

import synth
from paper_2210_04184_amd import nlpr

pytestmark = pytest.mark.gpu

CASES = [dict(p=8, q=8, L=3, Lh=1, d=2, blur_radius=1, K=0, Sw=1),
         dict(p=18, q=24, L=2, Lh=4, d=2, blur_radius=1, K=1, Sw=2),
         dict(p=24, q=36, L=31, Lh=3, d=3, blur_radius=2, K=1, Sw=1),
         dict(p=27, q=36, L=64, Lh=2, d=9, blur_radius=1, K=2, Sw=2),
         dict(p=36, q=48, L=65, Lh=2, d=2, blur_radius=1, K=1, Sw=1),
         dict(p=32, q=48, L=5, Lh=1, d=4, blur_radius=2, K=3, Sw=4),
         dict(p=24, q=24, L=5, Lh=2, d=4, blur_radius=1, K=4, Sw=5),
         dict(p=24, q=972, L=5, Lh=2, d=4, blur_radius=2, K=1, Sw=2),
         dict(p=256, q=256, L=44, Lh=1, d=4, blur_radius=1, K=1, Sw=1),
         dict(p=384, q=384, L=32, Lh=4, d=4, blur_radius=1, K=1, Sw=1),
         dict(p=512, q=512, L=18, Lh=2, d=4, blur_radius=1, K=2, Sw=1)]
FORMS = {"plain": {}, "graph": dict(flags=nlpr.GRAPH), "fused-S": dict(flags=nlpr.FUSED_S)}


def _scene(kw, seed=11):
    return synth.make_scene(synth.small_spec(iters=5, seed=seed, **kw))


def _solve(sc, flags, **over):
    plan = nlpr.Plan.from_scene(sc, flags, **over)
    Z, ws = plan.solve(torch.from_numpy(sc.Yl).cuda(), torch.from_numpy(sc.Yh).cuda())
    lam = [nlpr.REGION_LAMBDA2] if flags & nlpr.FUSED_S else [nlpr.REGION_LAMBDA1,
                                                              nlpr.REGION_LAMBDA2]
    return Z, plan.state_sigma(ws), [plan.region_view(ws, r) for r in lam]


@pytest.mark.parametrize("form", sorted(FORMS))
@pytest.mark.parametrize("kw", CASES, ids=lambda kw: f"{kw['p']}x{kw['q']}x{kw['L']}")
def test_one_launch_equals_two(kw, form):
    sc = _scene(kw)
    flags = FORMS[form].get("flags", 0)
    a = _solve(sc, flags)
    b = _solve(sc, (flags & ~nlpr.GRAPH) | nlpr.TIMING)
    assert torch.isfinite(a[0]).all()
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    for x, y in zip(a[2], b[2]):
        assert torch.equal(x, y)


def test_one_launch_equals_two_with_a_basis():
    sc = _scene(dict(p=24, q=36, L=12, Lh=2, d=4, blur_radius=2, K=1, Sw=2))
    E = np.linalg.qr(np.random.default_rng(5).standard_normal((12, 5)))[0].T
    E = np.ascontiguousarray(E, dtype=np.float32)
    a, b = _solve(sc, 0, E=E), _solve(sc, nlpr.TIMING, E=E)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])


@pytest.mark.parametrize("kw", [CASES[i] for i in (1, 2, 3, 5)],
                         ids=lambda kw: f"{kw['p']}x{kw['q']}x{kw['L']}")
def test_differentiated_solve(kw):
    """The forward pass that records checkpoints and branch codes gives the solve's bits."""
    sc = _scene(kw)
    plan = nlpr.Plan.from_scene(sc)
    Z = plan.forward(torch.from_numpy(sc.Yl).cuda(), torch.from_numpy(sc.Yh).cuda())[0]
    assert torch.equal(Z, _solve(sc, nlpr.TIMING)[0])
