"""A scene whose dual state the sweep keeps in the caches when it is solved alone, and streams when
it is solved in a batch with more state: same iterates, same decoded dual state, bit for bit; and
below the line, where the plain solve streams the values and the differentiated one caches them."""
import pytest
import torch

import synth
from paper_2210_04184_amd import nlpr

pytestmark = pytest.mark.gpu


def _inputs(sc):
    return torch.from_numpy(sc.Yl).cuda(), torch.from_numpy(sc.Yh).cuda()


def _scene(**kw):
    return synth.make_scene(synth.small_spec(**dict(dict(Lh=1, d=4, blur_radius=1, K=1, Sw=1, iters=5,
                                                         seed=9), **kw)))


@pytest.mark.parametrize("kw", [dict(p=128, q=128, L=33), dict(p=192, q=192, L=15)],
                         ids=["128x128x33", "192x192x15"])
def test_cached_alone_streamed_in_a_batch(kw):
    sc = _scene(**kw)
    plan = nlpr.Plan.from_scene(sc)
    Z, ws = plan.solve(*_inputs(sc))
    batch = nlpr.Batch.from_scenes([sc] * 6)
    ins = [_inputs(sc) for _ in range(6)]
    Zs, wsb = batch.solve([a for a, _ in ins], [b for _, b in ins])
    part = lambda i, r: (lambda o, n: wsb[o:o + n])(*batch.region(i, r))
    for i in (0, 5):
        assert torch.equal(Zs[i], Z)
        sig = plan.sigma_expand(part(i, nlpr.REGION_SIGMA).view(torch.float32),
                                part(i, nlpr.REGION_SIGMA_CODES),
                                part(i, nlpr.REGION_MU).view(torch.float32))
        assert torch.equal(sig, plan.state_sigma(ws))


@pytest.mark.parametrize("kw", [dict(p=24, q=36, L=5, Sw=2), dict(p=64, q=64, L=8, K=2, Sw=3),
                                dict(p=128, q=128, L=31)], ids=lambda kw: "{p}x{q}x{L}".format(**kw))
def test_differentiated_solve_equals_the_plain_one(kw):
    sc = _scene(**kw)
    plan = nlpr.Plan.from_scene(sc)
    assert torch.equal(plan.forward(*_inputs(sc))[0], plan.solve(*_inputs(sc))[0])
