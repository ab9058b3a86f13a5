"""What the host side launches, on the CPU: tests/c/host_launches.cpp runs the library on HIP
runtime functions of its own, which print each launch in place of making it."""
import os
import shutil
import subprocess
from collections import namedtuple

import pytest

from paper_2210_04184_amd import build, nlpr

HERE = os.path.dirname(os.path.abspath(__file__))
Launch = namedtuple("Launch", "phase kernel grid block lds limit table")


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    if not os.path.exists(nlpr.LIB_PATH) or not (shutil.which("hipcc") or
                                                 os.path.exists("/opt/rocm/bin/hipcc")):
        pytest.skip("needs libnlpr.so and hipcc")
    exe = str(tmp_path_factory.mktemp("host") / "host_launches")
    lib = os.path.dirname(nlpr.LIB_PATH)
    flags = [f for f in build.HIP_FLAGS if f not in ("-O3", "-fPIC")]
    res = subprocess.run([build.hipcc(), "--offload-host-only", "-x", "hip", *flags,
                          os.path.join(HERE, "c", "host_launches.cpp"), "-o", exe, "-L", lib,
                          "-lnlpr", "-Wl,-rpath," + lib], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr

    def go(n=1, p=24, q=36, L=3, Lh=1, d=2, r=1, K=1, Sw=1, iters=3, flags=0, more=()):
        """(launches, {phase: status})"""
        args = [exe, *map(str, (n, p, q, L, Lh, d, r, K, Sw, iters, flags)), *more]
        res = subprocess.run(args, capture_output=True, text=True, timeout=60)
        assert res.returncode == 0, res.stderr
        launches, status = [], {}
        for line in res.stdout.splitlines():
            f = line.split()
            if f[1] == "status":
                status[f[0]] = int(f[2])
            else:
                launches.append(Launch(f[0], f[1], *map(int, f[2:6]), f[6]))
        return launches, status
    return go


@pytest.mark.parametrize("n", [1, 2])
@pytest.mark.parametrize("kw", [dict(), dict(q=3888, K=0), dict(q=4096, K=0), dict(p=4096, q=24),
                                dict(p=4096, q=24, d=1, flags=nlpr.FUSED_S),
                                dict(p=1536, q=24, d=4, flags=nlpr.FUSED_S),
                                dict(q=972, K=4, Sw=8)],
                         ids=lambda kw: "-".join(f"{k}{v}" for k, v in kw.items()) or "small")
def test_dynamic_lds_is_within_each_kernels_limit(run, kw, n):
    launches, status = run(n=n, **kw)
    assert set(status.values()) == {nlpr.OK}
    assert {"create", "solve"} <= {x.phase for x in launches}
    assert [x for x in launches if x.lds > x.limit or x.limit > 160 * 1024] == []


@pytest.mark.parametrize("kw", [dict(), dict(K=4, Sw=2), dict(p=24, q=1536, L=2),
                                dict(p=36, q=48, flags=nlpr.STATE_IN)],
                         ids=["one launch", "two launches", "several items", "resumed"])
def test_sweeps_need_their_table(run, kw):
    """The sweep's items are in an order of their own, so its kernels index the table without a
    look: a launch without one is refused on the host, in every pass, before it is made."""
    launches, status = run(**kw)
    grad = kw.get("q", 0) <= 1024 and not kw.get("flags")   # else refused
    assert set(status.values()) == {nlpr.OK} and ("backward" in status) == grad
    sweeps = [x for x in launches if "sweep" in x.kernel]
    assert sweeps and {x.table for x in sweeps} == {"table"}
    launches, status = run(**kw, more=["no-table"])
    assert status.pop("create") == nlpr.OK
    assert set(status.values()) == {nlpr.ERR_HIP}
    assert not any("sweep" in x.kernel for x in launches)


@pytest.mark.parametrize("kw", [dict(p=96, q=64, L=31), dict(p=48, q=48, d=4, flags=nlpr.FUSED_S)],
                         ids=["plain", "fused-S"])
def test_tuner_times_the_order_that_the_solve_runs(run, kw):
    """The passes of the X-update run without a table in a solve of one scene, in the order that
    keeps neighbouring work items on one XCD; their shapes are tuned in the same order."""
    launches, _ = run(**kw)
    tables = {p: {x.table for x in launches if x.phase == p and "fft_" in x.kernel}
              for p in ("create", "solve")}
    assert tables == {"create": {"null"}, "solve": {"null"}}


@pytest.mark.parametrize("flags", [0, nlpr.FUSED_S], ids=["plain", "fused-S"])
def test_a_batch_is_made_without_timing_shapes_it_does_not_use(run, flags):
    """Scenes of a batch take the shapes of a rule: making one launches no pass of the X-update."""
    launches, status = run(n=3, p=48, q=36, d=4, flags=flags)
    assert set(status.values()) == {nlpr.OK}
    assert {x.phase for x in launches if "fft_" in x.kernel} == {"solve"}


@pytest.mark.parametrize("p,q,freq", [(8, 12, 16), (192, 324, 16), (256, 256, 64), (243, 324, 64),
                                      (1024, 96, 64)])
def test_denominator_variant(run, p, q, freq):
    """Frequencies per workgroup on both sides of the line, and workgroups for all of them."""
    launches, _ = run(p=p, q=q, d=1, iters=0)
    (den,) = [x for x in launches if "den_kernel" in x.kernel]
    assert f"den_kernelILi{freq}E" in den.kernel
    assert (den.grid - 1) * freq < q <= den.grid * freq and den.block == 256


@pytest.mark.parametrize("p,q,parts", [(8, 8, 4), (18, 108, 4), (48, 64, 4), (96, 96, 4),
                                       (324, 384, 4), (384, 384, 1)])
def test_p_update_covers_its_items_by_xcd(run, p, q, parts):
    """With several workgroups per work item of 256 pixels, workgroup b takes part b / 8 of one of
    eight items, on the XCD (b % 8) of the item's index: whole groups of eight are launched."""
    items = -(-p * q // 256)
    launches, _ = run(p=p, q=q, d=1, iters=2, flags=nlpr.TIMING)
    grids = {x.grid for x in launches if "pupdate_kernel" in x.kernel}
    assert grids == {items if parts == 1 else -(-items // 8) * 8 * parts}


def _policies(launches, phase):
    """Cache policies (last template argument) of the sweeps of a phase."""
    return {int(x.kernel.split("ELi")[-1].split("E")[0]) for x in launches
            if x.phase == phase and ("12sweep_kernel" in x.kernel or "sweep_pu_kernel" in x.kernel)}


@pytest.mark.parametrize("kw,solve,forward",
                         [(dict(p=64, q=64, L=8, K=2, Sw=3), 1, 0),           # 80 MB of state
                          (dict(p=128, q=128, L=31, K=1, Sw=1), 1, 0),        # 2^19 - 16384 pixel-bands
                          (dict(p=128, q=128, L=32, K=1, Sw=1), 0, 0),        # 2^19
                          (dict(p=96, q=96, L=8, K=2, Sw=3), 1, 0),           # 179 MB
                          (dict(p=192, q=192, L=8, K=2, Sw=2), 0, 0),         # 358 MB, below 2^19
                          (dict(p=64, q=64, L=8, K=3, Sw=5), 1, 1),           # 390 MB
                          (dict(p=256, q=256, L=37, K=1, Sw=1), 0, 0),        # 354 MB, above 2^19
                          (dict(p=256, q=256, L=124, K=1, Sw=1), 2, 2),       # 1.2 GB in 36 planes
                          (dict(p=128, q=128, L=32, K=1, Sw=1, n=4), 0, None),
                          (dict(p=128, q=128, L=32, K=1, Sw=1, n=6), 1, None)],
                         ids=lambda v: "-".join(map(str, v.values())) if isinstance(v, dict) else str(v))
def test_cache_policy_of_the_sweep(run, kw, solve, forward):
    """0: the dual state cached, 1: its values streamed, 2: all streamed, by its bytes, the planes
    per band and the pixel-bands of the whole batch; reverse mode by the bytes and planes alone."""
    launches, _ = run(d=1, iters=2, **kw)
    assert _policies(launches, "solve") == {solve}
    if forward is not None:
        assert _policies(launches, "forward") == {forward}
