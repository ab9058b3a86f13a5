"""Reverse mode over many iterations and at the edges of the shared launch of its two adjoints,
against the FP64 reference gradient at the reverse mode's bar of 1e-3 (see test_gpu_grad.py).

The descriptors of the iterations are written 32 at a time: the numbers of iterations lie on
both sides of one and two fillings.  These run without a window, where the iteration is smooth
in its inputs (with thresholds, FP32 and FP64 may take different branches somewhere in many
iterations, and the gradients then differ by right); with one, the forward pass of as many
iterations is compared with the plain solve bit for bit.  The shared launch: P-update workgroups
that end past the last pixel, tiles smaller than the exchange of shares, the most bands whose
threads hold them and one more, and guide bands of each register class."""
import pytest
import torch

from oracle import nlpr_grad as og
from oracle import nlpr_oracle as o
from paper_2210_04184_amd import nlpr
from test_gpu_grad import dev, gpu_grad, rel, scene

pytestmark = pytest.mark.gpu


def check(sc, T, over=None, okw=None):
    _, gYl, gYh, glam, grho, _ = gpu_grad(sc, **(over or {}))
    if T == 1 and okw:             # one X-update of the start: Y_h and lambda do not enter
        assert not gYh.any() and glam == 0.0 and abs(gYl).max() > 0.0
        return
    pr = o.Problem.from_scene(sc, **(okw or {}))
    ref = og.gradient(sc.Yl.astype("float64"), sc.Yh.astype("float64"), pr, T, sc.Z)
    assert rel(gYl, ref[1]) <= 1e-3
    assert rel(gYh, ref[2]) <= 1e-3
    assert glam == pytest.approx(ref[3], rel=1e-3, abs=1e-9)
    assert grho == pytest.approx(ref[4], rel=1e-3)


@pytest.mark.parametrize("T", [1, 2, 32, 33, 64, 65])
def test_iterations_past_one_filling(T):
    check(scene(16, 24, 3, 2, 4, 1, 1, 1, iters=T, seed=3), T, dict(Sw=0), dict(S=0))


@pytest.mark.parametrize("T", [1, 32, 33, 65])
def test_forward_of_many_iterations_equals_the_solve(T):
    sc = scene(16, 24, 3, 2, 4, 1, 1, 1, iters=T, seed=3)
    Z = nlpr.Plan.from_scene(sc).forward(dev(sc.Yl), dev(sc.Yh))[0]
    assert torch.equal(Z, nlpr.Plan.from_scene(sc).solve(dev(sc.Yl), dev(sc.Yh))[0])


@pytest.mark.parametrize("shape", [(8, 8, 3, 1, 2, 1, 0, 1), (18, 24, 2, 4, 2, 1, 1, 1),
                                   (12, 16, 32, 3, 4, 1, 1, 1), (12, 16, 33, 2, 4, 1, 1, 1),
                                   (12, 16, 6, 5, 4, 1, 1, 1), (16, 24, 2, 2, 2, 1, 3, 1),
                                   (18, 24, 2, 1, 2, 1, 4, 1)],
                         ids=lambda s: "x".join(map(str, s)))
def test_edges_of_the_shared_launch(shape):
    check(scene(*shape, iters=3), 3)
