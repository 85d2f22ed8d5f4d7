"""mt_run_static_scratch (the pass for callers that cannot allocate) against mt_run, through the C ABI, on the GPU."""
import os
import subprocess
import sys

import numpy as np
import pytest

from paper_2111_14255_amd import binding as B
from synth import GraphBuilder, zoo
from gpu_harness import Mix, assert_close

pytestmark = pytest.mark.gpu


def small_split_model(dtype="f16"):
    """Two 3x3 layers on a 4x4 map and a classifier: every convolution is split along its reduction."""
    g = GraphBuilder("small_split", dtype, 1, 4, 4, 1024)
    t = g.conv(0, 1024, 3, pad=1, bn=True)
    t = g.conv(t, 512, 3, pad=1, bn=True, res=-1)
    t = g.gap(t)
    g.fc(t, 100)
    return g.done()


def wide_split_model(dtype="f16"):
    """Split layers on a patch (its epilogue can apply the pooling behind it) and on three tiles, and a classifier."""
    g = GraphBuilder("wide_split", dtype, 1, 28, 28, 512)
    t = g.conv(0, 256, 3, pad=1, bn=True)
    t = g.maxpool(t, 2, 2)
    t = g.conv(t, 512, 5, pad=2, bn=True)
    t = g.conv(t, 512, 5, pad=2, bn=True)
    t = g.conv(t, 64, 7, stride=2, pad=3, bn=True)
    t = g.gap(t)
    g.fc(t, 100)
    return g.done()


def both_ways(mix, sched):
    """Outputs of mt_run and of mt_run_static_scratch under the same schedule (output buffers poisoned before each)."""
    ref, _ = mix.run(sched)
    outs = [mix.ctx.make_output(t) for t in range(len(mix.specs))]
    for o in outs:
        o.fill_(float("nan"))
    tm = mix.ctx.run_static_scratch(sched, mix.inputs, outs)
    got = [mix.ctx.output_to_numpy(t, o) for t, o in enumerate(outs)]
    return ref, got, tm


def split_forms(mix, tenant):
    """Kernels of the tenant's convolutions whose partial sums meet in a workspace."""
    forms = [mix.ctx.op_form(tenant, i) for i in range(mix.ctx.lens()[tenant])]
    return [f.name.decode() for f in forms if f.split_k > 1 and f.workspace_bytes > 0]


def test_static_scratch_pass_equals_mt_run_twice_in_a_row():
    # first call: two tenants with many split layers; second call, right after it: a smaller tenant set, so that the
    # array still holds the first call's partial sums and counter values where the second one works
    big = Mix([wide_split_model(), zoo.BUILDERS["mobilenetv2"]("f16", 1)], seed=911)
    small = Mix([small_split_model()], seed=912)
    try:
        assert split_forms(big, 0) == ["patch_64x64", "tile_64x32", "tile_64x64", "tile_64x16"]
        assert split_forms(small, 0) == ["tile_64x16", "tile_64x16"]
        sb = big.ctx.schedule([[2, 4], [20, 40]], 3)
        ss = small.ctx.sequential()
        ref_b, got_b, tm_b = both_ways(big, sb)
        ref_s, got_s, tm_s = both_ways(small, ss)
        for r, g in zip(ref_b + ref_s, got_b + got_s):
            assert np.isfinite(g).all()
            np.testing.assert_array_equal(g, r)                   # same kernels, same reduction order: same bits
        assert tm_b["n_launches"] == sum(big.ctx.lens()) and tm_b["makespan_ms"] > 0 and tm_s["makespan_ms"] > 0
        # and the pass is the forward pass: oracle parity of the small one
        for t, m in enumerate(small.specs):
            assert_close(got_s[t], small.oracle()[t], m.dtype, m.name)
        # once more in the other order, all-concurrent, with a fused-pair schedule on the big set
        ref_s2, got_s2, _ = both_ways(small, ss)
        sb2 = big.ctx.all_concurrent(flags=B.MT_SCHED_FUSE_EXPAND | B.MT_SCHED_FUSE_POOL)
        ref_b2, got_b2, _ = both_ways(big, sb2)
        for r, g in zip(ref_s2 + ref_b2, got_s2 + got_b2):
            np.testing.assert_array_equal(g, r)
        for a, b in zip(ref_b, ref_b2):
            np.testing.assert_array_equal(a, b)
    finally:
        big.close()
        small.close()


def layers_side_by_side(n, shape, k, win, stride):
    """n convolutions of one input, each with its own output, and a classifier behind the last."""
    g = GraphBuilder("side_by_side", "f16", *shape)
    t = [g.conv(0, k, win, stride, win // 2, bn=True) for _ in range(n)][-1]
    g.fc(g.gap(t), 10)
    return g.done()


def test_static_scratch_counts_the_workspaces_that_are_used():
    # VGG-16 splits two layers (6.5 MiB), ResNet-18 none: its rings need no workspace
    mix = Mix([zoo.BUILDERS["vgg16"]("f16", 1), zoo.resnet18("f16", 1)], seed=913)
    try:
        forms = [mix.ctx.op_form(t, i) for t in range(2) for i in range(mix.ctx.lens()[t])]
        assert 0 < sum(f.workspace_bytes for f in forms) < B.MT_STATIC_SCRATCH_BYTES / 2
        assert any(f.ring_waves for f in forms)
        ref, got, _ = both_ways(mix, mix.ctx.all_concurrent())
        for r, g in zip(ref, got):
            np.testing.assert_array_equal(g, r)
    finally:
        mix.close()


def test_large_workspaces_stay_in_the_arena():
    # 14.25 MiB in one layer of each tenant, 0.75 MiB in the other: three tenants would need 45 MiB of the array
    def net():
        g = GraphBuilder("large_split", "f16", 12, 14, 14, 512)
        t = g.conv(0, 512, 3, pad=1, bn=True)
        g.conv(t, 64, 7, stride=2, pad=3, bn=True)
        return g.done()
    mix = Mix([net(), net(), net()], seed=914)
    try:
        ctx = mix.ctx
        sizes = [ctx.op_form(0, i).workspace_bytes for i in range(2)]
        assert sizes[0] > B.MT_STATIC_SCRATCH_BYTES / 4 and 0 < sizes[1] < B.MT_STATIC_SCRATCH_BYTES / 16
        ref, _ = mix.run(ctx.sequential())
        for s in (ctx.all_concurrent(), ctx.schedule([[], [], []], 1, concurrency=[1], flags=B.MT_SCHED_COISSUE), ctx.schedule([[1]] * 3, 2)):
            for _ in range(2):
                _, got, _ = both_ways(mix, s)
                for r, g in zip(ref, got):
                    np.testing.assert_array_equal(g, r)
    finally:
        mix.close()


MEASURE = """
import sys
sys.path[:0] = [%r, %r]
import numpy as np
import torch
from paper_2111_14255_amd import binding as B
from synth import zoo
from gpu_harness import Mix
from test_zz_no_alloc import split_forms, wide_split_model
split = %r
mix = Mix([zoo.BUILDERS["mobilenetv2"]("f16", 1), wide_split_model() if split else zoo.resnet18("f16", 1)], seed=915)
assert bool(split_forms(mix, 1)) == split
outs = [mix.ctx.make_output(t) for t in range(2)]
keep, taken = [], []
for i in range(100):
    co = mix.ctx.schedule([[], []], 1, concurrency=[1 + i %% 2], flags=(B.MT_SCHED_FUSE_POOL, B.MT_SCHED_FUSE_EXPAND, B.MT_SCHED_TIME_TENANTS)[i %% 3])
    if i %% 5 == 4:
        mix.ctx.run_static_scratch(co, mix.inputs, outs)
        co.set_wave_priority([i %% 4, -1])
    keep.append(co)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    mix.ctx.run_static_scratch(co, mix.inputs, outs)
    torch.cuda.synchronize()
    taken.append(before - torch.cuda.mem_get_info()[0])
assert not any(taken), taken
assert all(np.isfinite(mix.ctx.output_to_numpy(t, outs[t])).all() for t in range(2))
print("no memory taken")
"""


@pytest.mark.parametrize("split", [False, True])
def test_the_call_takes_no_device_memory(split):
    """In a process of its own, from its first call on.  The arguments of a schedule's packets take some 45 KiB, and device memory
    is handed out 2 MiB at a time: these many schedules take several such pieces, none of them in a call."""
    here = os.path.dirname(os.path.abspath(__file__))
    r = subprocess.run([sys.executable, "-c", MEASURE % (os.path.dirname(here), here, split)], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "no memory taken" in r.stdout, r.stdout + r.stderr


def test_static_scratch_limits_and_flags():
    # five split layers of 3.25 MiB each: more than the array holds
    mix = Mix([layers_side_by_side(5, (1, 28, 28, 512), 256, 3, 1), zoo.BUILDERS["tinyC"]("f16", 1)], seed=913)
    try:
        assert sum(mix.ctx.op_form(0, i).workspace_bytes for i in range(5)) > B.MT_STATIC_SCRATCH_BYTES
        outs = [mix.ctx.make_output(t) for t in range(2)]
        s = mix.ctx.sequential()
        with pytest.raises(B.MtError) as ei:
            mix.ctx.run_static_scratch(s, mix.inputs, outs)
        assert ei.value.code == B.MT_ERR_OUT_OF_MEMORY and str(B.MT_STATIC_SCRATCH_BYTES) in str(ei.value)
        for flags in (B.MT_SCHED_GRAPH, B.MT_SCHED_PARALLEL_ISSUE, B.MT_SCHED_STREAM_GRAPHS):
            sg = mix.ctx.all_concurrent(flags=flags)
            with pytest.raises(B.MtError) as ei:
                mix.ctx.run_static_scratch(sg, mix.inputs, outs)
            assert ei.value.code == B.MT_ERR_INVALID_ARG
        mix.ctx.run(s, mix.inputs, outs)                          # the ordinary pass still works after the refusals
        assert np.isfinite(mix.ctx.output_to_numpy(0, outs[0])).all()
    finally:
        mix.close()
