"""The X-update at widths whose row lines, with their padding, take more LDS than the default limit
of a launch (3888 and 4096 points), against float64 at the bound of test_gpu_fft.py; alone and as
scenes of a batch, whose row passes have another shape."""
import numpy as np
import pytest
import torch

import synth
from paper_2210_04184_amd import nlpr
from test_gpu_fft import test_solve_matches_float64 as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,q,L", [(8, 3888, 1), (9, 3888, 3), (12, 4096, 2)])
def test_wide_rows(p, q, L):
    check(p, q, L)


@pytest.mark.parametrize("q", [3888, 4096])
def test_wide_rows_in_a_batch(q):
    scenes = [synth.make_scene(synth.small_spec(p=8, q=w, L=2, Lh=1, d=2, blur_radius=1, K=0, Sw=1,
                                                iters=2, seed=w)) for w in (q, 48)]
    ins = [(torch.from_numpy(s.Yl).cuda(), torch.from_numpy(s.Yh).cuda()) for s in scenes]
    Zs, _ = nlpr.Batch.from_scenes(scenes).solve([a for a, _ in ins], [b for _, b in ins])
    for sc, (Yl, Yh), Z in zip(scenes, ins, Zs):
        assert np.isfinite(Z.cpu().numpy()).all()
        assert torch.equal(Z, nlpr.Plan.from_scene(sc).solve(Yl, Yh)[0])
