"""The packed storage of the coded dual state, slot by slot.  The runs of a sweep end on whole
64-byte blocks, but never past the capacity of their segment, where the next segment or plane
begins.  The region and a guard behind it are filled with a pattern; after each sweep the open
items of every segment are counted from the code bytes, and every slot past the longest run so far
(rounded up to its 64-byte block, at most the segment's items) still has to hold the pattern.  The
same for Sigma'' of the reverse pass, whose stored items follow from the branch codes.  The decoded
state is compared with the same updates in float64."""
import numpy as np
import pytest
import torch

import synth
from paper_2210_04184_amd import nlpr

PATTERN = 0x7fc0dead
GUARD = 1 << 12                   # slots behind the region

# partial tiles, segments of fewer than 64 items, planes that start inside a 64-byte block, waves
# without an item; two and four items per thread (no reverse pass)
SHAPES = [dict(p=8, q=8, L=2, K=0, Sw=1), dict(p=9, q=12, L=3, K=1, Sw=1),
          dict(p=24, q=36, L=5, K=1, Sw=2), dict(p=18, q=108, L=3, K=2, Sw=1),
          dict(p=16, q=384, L=4, K=1, Sw=1), dict(p=27, q=972, L=2, K=1, Sw=1),
          dict(p=18, q=24, L=2, K=4, Sw=1), dict(p=9, q=1536, L=2, K=1, Sw=1),
          dict(p=8, q=3888, L=1, K=0, Sw=2)]
ids = lambda kw: "{p}x{q}x{L}-K{K}".format(**kw)


def run_ends(stored, at):
    """Slots that a sweep may have written, per (plane, item).  stored: [planes][items per plane]
    bool; at: slot of the region's first item in its 64-byte block."""
    planes, items = stored.shape
    slot = torch.arange(items, device=stored.device)
    start = slot // 64 * 64
    seg = torch.zeros(planes, -(-items // 64), dtype=torch.long, device=stored.device)
    seg.index_add_(1, slot // 64, stored.long())
    first = torch.arange(planes, device=stored.device)[:, None] * items + torch.arange(
        seg.shape[1], device=stored.device) * 64 + at          # each segment's first slot
    end = (first + seg + 3) // 4 * 4 - first                   # its run's end, by whole blocks
    end = torch.where(seg > 0, end, torch.zeros_like(end))
    return slot - start < end[:, slot // 64]


def strays(slots, allowed):
    """Slots outside the allowed ones, the guard among them, that do not hold the pattern."""
    held = (slots == PATTERN).all(dim=-1)
    n = allowed.numel()
    return int((~held[:n] & ~allowed.flatten()).sum()) + int((~held[n:]).sum())


@pytest.mark.parametrize("cap", [True, False])
@pytest.mark.parametrize("at", [0, 1, 3])
def test_the_count_sees_a_run_past_its_segment(at, cap):
    """The check itself, on a simulated store: a run of 35 slots in a plane of 36, written up to the
    end of its 64-byte block, with the plane's capacity as its cap or without."""
    stored = torch.zeros(3, 36, dtype=torch.bool)
    stored[0, :35] = True
    end = (at + 35 + 3) // 4 * 4 - at               # 36, 35 and 37
    slots = torch.full((3 * 36 + 8, 4), PATTERN, dtype=torch.int32)
    slots[:min(end, 36) if cap else end] = 0
    assert strays(slots, run_ends(stored, at)) == (0 if cap else max(0, end - 36))


def _scene(kw, iters):
    return synth.make_scene(synth.small_spec(Lh=1, d=1, blur_radius=1, iters=iters, seed=3, **kw))


def _filled(nfloats):
    return torch.full((nfloats // 4 + GUARD, 4), PATTERN, dtype=torch.int32, device="cuda")


@pytest.mark.gpu
@pytest.mark.parametrize("kw", SHAPES, ids=ids)
def test_sweeps_write_their_runs_only(kw):
    sc = _scene(kw, 1)
    plan = nlpr.Plan.from_scene(sc)
    inf = plan.info()
    p, q, L, K = kw["p"], kw["q"], kw["L"], kw["K"]
    gen = torch.Generator(device="cuda").manual_seed(5)
    rnd = lambda *s: torch.rand(*s, generator=gen, device="cuda")
    mu = 0.5 * rnd(inf.npairs, p, q)
    ws = plan.alloc_workspace()
    codes = plan.region_bytes(ws, nlpr.REGION_SIGMA_CODES)
    codes.zero_()                   # lanes past a partial tile write none
    slots = _filled(inf.sigma_elems)
    assert slots.data_ptr() % 64 == 0
    sig = slots.view(torch.float32).flatten()[:inf.sigma_elems]
    items = inf.tile_rows * q // 4
    allowed = torch.zeros(inf.sigma_elems // 4 // items, items, dtype=torch.bool, device="cuda")
    S = torch.zeros(inf.npairs, inf.npatch, L, p, q, dtype=torch.float64, device="cuda")
    X, C = torch.empty(L, p, q, device="cuda"), torch.empty(L, p, q, device="cuda")
    for i, scale in enumerate((0.3, 1.5, 0.1)):      # mostly open, mostly on the threshold, open
        X.copy_(scale * rnd(L, p, q))
        plan.stage(nlpr.STAGE_SWEEP if i else nlpr.STAGE_SWEEP_FIRST, [X, mu, sig, C, ws])
        stored = codes.view(-1, items) >= 16
        allowed |= run_ends(stored, 0)
        assert bool(stored.any()) and strays(slots, allowed) == 0
        for n, t in enumerate(plan.half_window()):
            g = X.double() - torch.roll(X.double(), t, (-2, -1))
            for k in range(inf.npatch):
                k1, k2 = k // (2 * K + 1) - K, k % (2 * K + 1) - K
                thr = torch.roll(mu[n].double(), (-k1, -k2), (-2, -1))
                S[n, k] = -torch.maximum(torch.minimum(g - S[n, k], thr), -thr)
        got = plan.sigma_expand(sig, codes, mu).double()
        # two float32 roundings of values up to 2 max|X| + max mu in each sweep (clip adds none)
        assert float((got - S).abs().max()) <= 2.0 ** -23 * (i + 1) * (3.0 + 0.5)


@pytest.mark.gpu
@pytest.mark.parametrize("T", [2, 3])
@pytest.mark.parametrize("kw", SHAPES[:7], ids=ids)
def test_reverse_sweeps_write_their_runs_only(kw, T):
    sc = _scene(kw, T)
    plan = nlpr.Plan.from_scene(sc)
    inf = plan.info()
    p, q, L = kw["p"], kw["q"], kw["L"]
    Yl, Yh, dZ = (torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()
                  for a in (sc.Yl, sc.Yh, sc.Z))
    ckb, gwsb = plan.grad_sizes()
    ck = torch.zeros(ckb, dtype=torch.uint8, device="cuda")
    gws = torch.full((gwsb // 4,), PATTERN, dtype=torch.int32, device="cuda")
    _, ws, _ = plan.forward(Yl, Yh, ck=ck)
    plan.backward(Yl, Yh, dZ, ws, ck, gws=gws.view(torch.uint8))
    plane = -(-4 * L * p * q // 256) * 256
    nbytes = inf.sigma_elems // 4
    items = inf.tile_rows * q // 4
    # the checkpoints' branch codes follow the planes of X, B X and both Lambda
    at = 4 * (T - 1) * plane
    allowed, step = 0, -(-nbytes // 256) * 256
    for t in range(T - 1):
        b = ck[at + t * step:at + t * step + nbytes].view(-1, items)
        stored = ((b | (b >> 1)) & 0x55) != 0x55
        # lanes past a partial tile have no code (here 0) and store nothing
        rows = torch.arange(items, device="cuda") // (q // 4)
        tile = torch.arange(b.shape[0], device="cuda") // (inf.npairs * inf.npatch) % inf.ntiles
        stored &= rows < (p - tile * inf.tile_rows)[:, None]
        allowed = allowed | run_ends(stored, 0)
    # Sigma'' follows seven planes of the gradient workspace
    sig = gws[7 * plane // 4:7 * plane // 4 + inf.sigma_elems].view(-1, 4)
    assert gws.data_ptr() % 64 == 0 and bool(allowed.any())
    assert strays(sig, allowed) == 0
    first = allowed.flatten().nonzero()[0]
    assert not bool((sig[first] == PATTERN).all())    # the region is where it is looked for
