"""Threshold branches at thresholds that are not a number.  A NaN in Y_h makes every threshold
within reach of its pixel a NaN; an element there takes the branch of a threshold of 0, |V| < mu
being false for both, whatever the sign of the NaN.  An infinity in the same pixel makes the same
thresholds 0 (exp(-inf)), and up to the first sweep the iterates do not depend on Y_h, so after
two iterations the gradient with respect to Y_l, which is linear in dZ given the branches, must be
the same for both, bit for bit; after three too, V being a NaN everywhere in the second sweep."""
import pytest
import torch

from paper_2210_04184_amd import nlpr
from test_gpu_grad import dev, scene

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [2, 3])
@pytest.mark.parametrize("shape", [(16, 64, 4, 1, 2, 2, 0, 1), (24, 36, 5, 2, 4, 2, 1, 2),
                                   (32, 32, 6, 3, 4, 2, 2, 1), (24, 36, 3, 1, 4, 1, 4, 1)],
                         ids=lambda s: "x".join(map(str, s)))
def test_nan_thresholds_take_the_branch_of_zero(shape, T):
    sc = scene(*shape, iters=T)
    Yl, dZ = dev(sc.Yl), dev(sc.Z)
    grads = []
    for bad in (float("inf"), float("nan")):
        Yh = dev(sc.Yh)
        Yh[0, 5, 7] = bad
        plan = nlpr.Plan.from_scene(sc)
        _, ws, ck = plan.forward(Yl, Yh)
        mu = plan.region_view(ws, nlpr.REGION_MU)
        assert bool((mu.isnan() if bad != bad else mu == 0).any())
        grads.append(plan.backward(Yl, Yh, dZ, ws, ck)[0])
    assert bool(torch.isfinite(grads[0]).all()) and bool(grads[0].any())
    assert torch.equal(*grads)
