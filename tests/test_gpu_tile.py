"""The tile kernels that copy their operands from memory to LDS directly: every tile, way to gather an im2col row and patch
form, with ragged pixel and channel counts, split reductions, residual, channel offsets and the pooled epilogue, against a
plain fp32 convolution on the CPU."""
import re

import numpy as np
import pytest
import torch
import torch.nn.functional as F

from synth import GraphBuilder
from oracle import forward as OF
from oracle import ops as oops
from gpu_harness import Mix, assert_close
from paper_2111_14255_amd import binding as B

pytestmark = pytest.mark.gpu

CASES = [
    # name (the form the sizes lead to, "tile_" left out, and the split), n, h, w, c, k, window, stride, pad
    ("64x64_point", 3, 77, 91, 128, 136, 1, 1, 0),
    ("128x64_point_ragged_channels", 2, 90, 91, 192, 520, 1, 1, 0),
    ("128x128_point", 3, 70, 70, 320, 200, 1, 1, 0),
    ("64x32_point", 1, 60, 60, 512, 72, 1, 1, 0),
    ("64x16_point_half_stage", 1, 9, 13, 320, 520, 1, 1, 0),
    ("64x64_deep_tap_stride2", 5, 56, 57, 64, 200, 3, 2, 1),
    ("128x128_tap", 1, 121, 130, 64, 256, 3, 1, 1),
    ("64x32_tap", 1, 60, 62, 128, 128, 3, 1, 1),
    ("64x16_tap_5x5_wider_than_padding", 1, 41, 39, 64, 96, 5, 1, 2),
    ("64x16_tap_split8_stride2", 2, 9, 9, 1024, 100, 3, 2, 1),
    ("64x32_tap_split3", 1, 46, 46, 256, 64, 3, 1, 1),
    ("64x64_chunk_split3_5x5", 1, 66, 66, 72, 24, 5, 1, 2),
    ("128x64_chunk_split3_5x5", 6, 27, 27, 96, 256, 5, 1, 2),
    ("128x128_tap_split3_stride2", 12, 56, 56, 256, 256, 3, 2, 1),
    ("ring_32x16_tap_5x5", 1, 35, 33, 64, 96, 5, 1, 2),
    ("ring_16x16_tap_stride2", 2, 31, 31, 192, 100, 3, 2, 1),
    ("128x64_chunk_c72", 4, 60, 60, 72, 260, 3, 1, 1),
    ("64x16_chunk_c8_15x3", 1, 50, 50, 8, 24, (15, 3), 1, (7, 1)),
    ("ring_16x16_chunk_c8_15x3", 1, 30, 30, 8, 24, (15, 3), 1, (7, 1)),
    ("64x16_chunk_c24_unaligned_channels", 2, 13, 11, 24, 67, 3, 1, 1),
    ("64x16_one_pixel_split8", 9, 1, 1, 9216, 1000, 1, 1, 0),
    ("ring_16x16_one_pixel", 9, 1, 1, 4096, 520, 1, 1, 0),
    # windows of more than 15 rows or columns
    ("64x16_far_1x20_even_window", 3, 17, 9, 16, 32, (1, 20), 1, (0, 10)),
    ("64x16_far_split8_17x17_wider_than_the_map", 1, 8, 8, 64, 72, 17, 1, 8),
    ("64x16_far_split8_18x3_stride2", 1, 20, 30, 72, 100, (18, 3), 2, (9, 1)),
    ("64x32_far_1x17", 1, 60, 60, 64, 72, (1, 17), 1, (0, 8)),
    ("64x32_far_split4_17x1", 1, 20, 20, 256, 256, (17, 1), 1, (8, 0)),
    ("64x64_far_1x16_c8", 4, 80, 80, 8, 64, (1, 16), 1, (0, 8)),
    ("64x64_far_16x5_c24", 2, 40, 40, 24, 136, (16, 5), 1, (8, 2)),
    ("64x64_far_split7_1x31", 1, 48, 48, 128, 64, (1, 31), 1, (0, 15)),
    ("128x64_far_3x16_c8", 2, 70, 70, 8, 72, (3, 16), 1, (1, 8)),
    ("128x64_far_split3_1x31_ragged_channels", 6, 40, 40, 64, 124, (1, 31), 1, (0, 15)),
    ("patch_64x64_panel_of_one_column", 1, 62, 61, 192, 136, 3, 1, 1),
    ("patch_64x64_tiles_span_images", 40, 7, 7, 64, 320, 3, 1, 1),
    ("patch_64x64_split4", 1, 28, 28, 512, 256, 3, 1, 1),
    ("patch_64x32_odd_map", 2, 17, 17, 192, 512, 3, 1, 1),
    ("patch_128x64_wide_panel", 1, 100, 66, 128, 256, 3, 1, 1),
    ("patch_128x128_last_panel_partial", 2, 66, 97, 128, 256, 3, 1, 1),
    ("patch_128x128_split3", 3, 28, 28, 512, 512, 3, 1, 1),
    ("patch_128x256", 2, 112, 112, 64, 256, 3, 1, 1),
    ("patch_128x256_split3_tiles_span_images", 6, 28, 28, 384, 512, 3, 1, 1),
    ("128x64_split3_one_pixel_maps_no_patch_holds_the_batch", 300, 1, 1, 512, 2048, 3, 1, 1),
    ("128x64_2x2_maps_only_a_narrow_patch_fits", 700, 2, 2, 256, 512, 3, 1, 1),
    ("64x64_two_pixel_maps_no_patch_holds_the_batch", 800, 1, 2, 256, 512, 3, 1, 1),
]
ACT = {"none": lambda v: v, "relu": torch.relu, "relu6": lambda v: v.clamp(0, 6)}


def conv_ref(x, p, stride, pad, act, dtype):
    """x: fp32 NHWC values of the storage type; the stored result as fp32 NHWC."""
    w = torch.from_numpy(np.ascontiguousarray(p[0])).permute(0, 3, 1, 2)
    y = F.conv2d(torch.from_numpy(x).permute(0, 3, 1, 2), w, torch.from_numpy(p[1]), stride, pad)
    return y, ACT[act]


def check_form(ctx, name):
    want = re.match(r"(patch_|ring_)?(\d+x\d+)", name)
    split = re.search(r"split(\d+)", name)
    form = ctx.op_form(0, 0)
    assert form.name.decode() == (want.group(1) or "tile_") + want.group(2)
    assert form.split_k == (int(split.group(1)) if split else 1)
    assert (form.workspace_bytes > 0) == (form.split_k > 1)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("name,n,h,w,c,k,win,stride,pad", CASES, ids=[c[0] for c in CASES])
def test_tile_kernels(name, n, h, w, c, k, win, stride, pad, dtype):
    g = GraphBuilder("t", dtype, n, h, w, c)
    a = g.conv(0, k, win, stride, pad, act="relu6", bn=True)
    d = g.new_tensor()                                   # the same convolution with a residual, written at a channel offset
    off = 8 if k % 8 == 0 else 3
    g.conv(0, k, win, stride, pad, act="relu", bn=True, res=a, dst=d, c_off=off, c_tot=k + off)
    g.conv(0, off, win, stride, pad, act="none", dst=d, c_off=0, c_tot=k + off)
    spec = g.done()
    print("case", name, dtype, flush=True)
    mix = Mix([spec], seed=37)
    try:
        check_form(mix.ctx, name)
        got, _ = mix.run(mix.ctx.sequential())
        x = oops.round_array(mix.x[0], dtype)
        p = OF.prepare_params(spec, mix.raw[0])
        y0, act = conv_ref(x, p[0], stride, pad, "relu6", dtype)
        t0 = oops.round_array(act(y0).permute(0, 2, 3, 1).contiguous().numpy(), dtype)
        y1, act = conv_ref(x, p[1], stride, pad, "relu", dtype)
        t1 = act(y1.permute(0, 2, 3, 1) + torch.from_numpy(t0))
        y2, _ = conv_ref(x, p[2], stride, pad, "none", dtype)
        ref = torch.cat([y2.permute(0, 2, 3, 1), t1], dim=3).numpy()
        read = mix.ctx.read_tensor(0, a, t0.shape)
        assert_close(read.astype(np.float32), t0, dtype, name)
        assert_close(got[0], ref.reshape(n, -1), dtype, name)
    finally:
        mix.close()


POOLED = [
    # name, n, h, w, c, k
    ("patch_64x64_split3", 1, 28, 28, 384, 384),
    ("patch_64x64_even_panel", 6, 30, 28, 128, 136),
    ("patch_64x32", 1, 28, 28, 192, 384),
    ("patch_128x64", 3, 60, 62, 192, 128),
    ("patch_128x128", 4, 56, 56, 128, 256),
    ("patch_128x256", 2, 112, 112, 64, 256),
    ("128x64_tap", 4, 64, 64, 64, 128),
    ("64x32_tap", 1, 60, 62, 128, 128),
    ("64x16_tap_split8", 1, 6, 6, 1536, 264),
]


@pytest.mark.parametrize("name,n,h,w,c,k", POOLED, ids=[c[0] for c in POOLED])
def test_pooled_epilogue_of_the_tile_kernels(name, n, h, w, c, k):
    g = GraphBuilder("t", "bf16", n, h, w, c)
    a = g.conv(0, k, 3, 1, 1, act="relu", bn=True)
    pl = g.maxpool(a, 2, 2, 0)
    g.gap(pl)
    spec = g.done()
    print("case", name, flush=True)
    mix = Mix([spec], seed=41)
    try:
        ctx = mix.ctx
        check_form(ctx, name)
        shape = (n, h // 2, w // 2, k)
        _, tm = mix.run(ctx.sequential(flags=B.MT_SCHED_FUSE_POOL))
        assert tm["n_fused"] == 1
        fused = ctx.read_tensor(0, pl, shape)
        _, tm = mix.run(ctx.sequential())
        assert tm["n_fused"] == 0
        np.testing.assert_array_equal(fused.view(np.uint32), ctx.read_tensor(0, pl, shape).view(np.uint32))
        y, act = conv_ref(oops.round_array(mix.x[0], "bf16"), OF.prepare_params(spec, mix.raw[0])[0], 1, 1, "relu", "bf16")
        ref = F.max_pool2d(act(y), 2).permute(0, 2, 3, 1).contiguous().numpy()
        assert_close(fused, ref, "bf16", name)
    finally:
        mix.close()


def test_patch_does_not_carry_non_finite_pixels_into_foreign_windows():
    """A patch holds rows of two images with an empty row between them and the columns beside its panel."""
    n, h, w, c, k = 2, 60, 62, 192, 128
    g = GraphBuilder("t", "bf16", n, h, w, c)
    g.conv(0, k, 3, 1, 1, act="none", bn=False)
    spec = g.done()
    mix = Mix([spec], seed=43)
    try:
        x = mix.x[0]
        for (i, r, q) in ((0, h - 1, 5), (0, 7, w - 1), (1, 0, 15), (1, 30, 16), (1, 31, 0)):
            x[i, r, q, 9] = np.nan
        mix.inputs[0] = mix.ctx.make_input(0, x)
        got, _ = mix.run(mix.ctx.sequential())
        y, _ = conv_ref(oops.round_array(x, "bf16"), OF.prepare_params(spec, mix.raw[0])[0], 1, 1, "none", "bf16")
        ref = y.permute(0, 2, 3, 1).contiguous().numpy().reshape(n, -1)
        bad = ~np.isfinite(ref)
        assert bad.any() and not bad.all()
        assert np.array_equal(~np.isfinite(got[0]), bad)
        scale = float(np.abs(ref[~bad]).max())
        assert float(np.abs(got[0][~bad] - ref[~bad]).max()) <= 2e-2 * scale
    finally:
        mix.close()


def test_far_windows_pooled_co_issued_and_beside_non_finite_pixels():
    """Windows of more than 15 rows or columns: the pooled epilogue and the launch of two tenants keep the bits, and a pixel that
    is not finite reaches the windows that hold it only."""
    n, h, w, c, k, win, pad = 2, 20, 22, 24, 72, (17, 4), (8, 2)
    g = GraphBuilder("far", "bf16", n, h, w, c)
    a = g.conv(0, k, win, 1, pad, act="none", bn=False)
    spec = g.done()
    g = GraphBuilder("far_pooled", "bf16", n, h, w, c)
    a = g.conv(0, k, win, 1, (8, 1), act="relu", bn=True)
    b = g.conv(a, 40, (1, 18), 1, (0, 9), act="relu", bn=True)
    pl = g.maxpool(b, 2, 2, 0)
    pooled = g.done()
    mix = Mix([spec, spec, pooled], seed=44)
    try:
        ctx = mix.ctx
        assert ctx.op_form(0, 0).name.startswith(b"tile_") and ctx.op_form(2, 1).name.startswith(b"tile_")
        x = mix.x[0]
        for (i, r, q) in ((0, h - 1, 5), (0, 3, w - 1), (1, 0, 9), (1, 12, 0)):
            x[i, r, q, 9] = np.nan
        mix.inputs[0] = ctx.make_input(0, x)
        plain, tm = mix.run(ctx.sequential())
        assert tm["n_fused"] == 0
        for flags, fused in ((B.MT_SCHED_COISSUE, 1), (B.MT_SCHED_FUSE_POOL, 1), (B.MT_SCHED_COISSUE | B.MT_SCHED_FUSE_POOL, 2)):
            got, tm = mix.run(ctx.schedule([[], [], []], 1, concurrency=[1], flags=flags))
            assert tm["n_fused"] == fused
            for p, q in zip(plain, got):
                np.testing.assert_array_equal(p, q)
        for t in range(3):
            xs = oops.round_array(mix.x[t], "bf16")
            p = OF.prepare_params(mix.specs[t], mix.raw[t])
            if t < 2:
                ref = conv_ref(xs, p[0], 1, pad, "none", "bf16")[0].permute(0, 2, 3, 1).contiguous().numpy()
            else:
                y, act = conv_ref(xs, p[0], 1, (8, 1), "relu", "bf16")
                y, act = conv_ref(oops.round_array(act(y).permute(0, 2, 3, 1).contiguous().numpy(), "bf16"), p[1], 1, (0, 9), "relu", "bf16")
                ref = F.max_pool2d(act(y), 2).permute(0, 2, 3, 1).contiguous().numpy()
            ref = ref.reshape(n, -1)
            bad = ~np.isfinite(ref)
            assert (bad.any() and not bad.all()) == (t == 0)
            assert np.array_equal(~np.isfinite(plain[t]), bad)
            assert float(np.abs(plain[t][~bad] - ref[~bad]).max()) <= 2e-2 * float(np.abs(ref[~bad]).max())
    finally:
        mix.close()


@pytest.mark.parametrize("name,n,h,w,c,k,win,stride,pad", [
    ("128x64_one_stage", 16, 28, 28, 64, 512, 1, 2, 0), ("128x128_two_stages", 16, 14, 14, 128, 1024, 1, 1, 0), ("128x64_three_stages", 15, 14, 13, 192, 520, 1, 1, 0),
    ("128x128_four_stages", 16, 14, 14, 256, 1024, 1, 1, 0), ("128x64_five_stages", 16, 14, 14, 320, 512, 1, 1, 0), ("128x128_chunk_ragged", 16, 28, 27, 72, 252, 3, 1, 1)])
def test_a_launch_that_has_the_chip_to_itself_keeps_the_bits(name, n, h, w, c, k, win, stride, pad):
    """The widest tiles stage more of the reduction ahead when nothing else runs: alone, beside another tenant, and on new buffers."""
    g = GraphBuilder("t", "bf16", n, h, w, c)
    g.conv(0, k, win, stride, pad, act="relu", bn=True)
    spec = g.done()
    print("case", name, flush=True)
    mix = Mix([spec, spec], seed=45)
    try:
        ctx = mix.ctx
        check_form(ctx, name)
        alone = ctx.schedule([[], []], 1, concurrency=[1])
        both = ctx.all_concurrent()
        assert alone.launch_forms() == (0, 0)            # nothing has run yet
        first, _ = mix.run(alone)
        beside, _ = mix.run(both)
        again, _ = mix.run(alone)                        # other output buffers: the arguments are written again
        assert alone.launch_forms() == (0, 2) and both.launch_forms() == (0, 0)
        for p, q, r in zip(first, beside, again):
            assert np.isfinite(p).all()
            np.testing.assert_array_equal(p, q)
            np.testing.assert_array_equal(p, r)
    finally:
        mix.close()


@pytest.mark.parametrize("dtype,share", [("bf16", 32), ("f16", 40), ("bf16", 8)])
def test_workgroups_that_walk_several_tiles_keep_the_bits(dtype, share):
    """More queues with a share of the units than dispatch pipes: launches larger than a share holds at once are walked by as many
    workgroups as fit.  Every form that has such a kernel, tiles that do not divide evenly among them, and a split reduction."""
    layers = [("128x128_tap_split3_stride2", 12, 56, 56, 256, 256, 3, 2, 1), ("128x64_c192", 15, 14, 13, 192, 520, 1, 1, 0), ("64x64_point", 3, 77, 91, 128, 136, 1, 1, 0),
              ("64x64_deep_tap_stride2", 5, 56, 57, 64, 200, 3, 2, 1), ("64x32_point", 1, 60, 60, 512, 72, 1, 1, 0), ("128x128_point", 3, 70, 70, 320, 200, 1, 1, 0),
              ("patch_64x64_split4", 1, 28, 28, 512, 256, 3, 1, 1), ("patch_64x32_odd_map", 2, 17, 17, 192, 512, 3, 1, 1), ("patch_128x64_wide_panel", 1, 100, 66, 128, 256, 3, 1, 1),
              ("patch_128x128_last_panel_partial", 2, 66, 97, 128, 256, 3, 1, 1), ("patch_128x256", 2, 112, 112, 64, 256, 3, 1, 1)]
    specs = []
    for name, n, h, w, c, k, win, stride, pad in layers:
        g = GraphBuilder(name, dtype, n, h, w, c)
        g.conv(0, k, win, stride, pad, act="relu", bn=True)
        specs.append(g.done())
    g = GraphBuilder("resident", dtype, 5, 112, 112, 64)                 # the resident-filter and first-layer kernels walk by themselves
    g.conv(g.conv(0, 256, 1, 1, 0, act="relu", bn=True), 64, 1, 1, 0, act="none", bn=True)
    g.conv(0, 64, 3, 1, 1, act="relu", bn=True)
    specs.append(g.done())
    g = GraphBuilder("first", dtype, 6, 224, 224, 3)
    g.conv(0, 64, 7, 2, 3, act="relu", bn=True)
    specs.append(g.done())
    for first in range(0, len(specs), 8):
        group = specs[first:first + 8] if len(specs) - first >= 8 else specs[-8:]
        mix = Mix(group, seed=46)
        try:
            ctx = mix.ctx
            for t, spec in enumerate(group):
                if re.match(r"(patch_)?\d+x", spec.name):
                    assert ctx.op_form(t, 0).name.decode().endswith(re.search(r"\d+x\d+", spec.name).group(0))
            print("case", dtype, share, [s.name for s in group], flush=True)
            alone, four = ctx.sequential(), ctx.schedule([[] for _ in group], 1, cu_share=[share] * 4 + [0] * (len(group) - 4), concurrency=[4])
            plain, _ = mix.run(alone)
            mix.run(four)                                # four queues have a dispatch pipe each
            assert alone.launch_forms()[0] == 0 and four.launch_forms() == (0, 0)
            shared = ctx.schedule([[] for _ in group], 1, cu_share=[share] * len(group))
            for _ in range(2):
                got, _ = mix.run(shared)
                assert shared.launch_forms() == (sum(len(spec.ops) for spec in group), 0)      # all of them are larger than their share
                for p, q in zip(plain, got):
                    assert np.isfinite(p).all()
                    np.testing.assert_array_equal(p, q)
        finally:
            mix.close()


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_walking_workgroups_with_residuals_pooling_and_channels_in_fours(dtype):
    """The epilogues of launches cut to a share: a residual, channel counts that are multiples of 4 only, 2x2 max pooling, a split reduction that pools; and
    a fused 1x1 + depthwise pair, which is never cut, beside them."""
    residual = [("tile_128x128", 3, 70, 70, 320, 196, 1), ("tile_128x64", 15, 14, 13, 192, 516, 1), ("tile_64x64", 3, 77, 91, 128, 140, 1),
                ("tile_64x32", 1, 60, 60, 512, 76, 1), ("patch_64x32", 1, 28, 28, 256, 508, 3), ("patch_128x128", 2, 66, 98, 128, 252, 3)]
    pooled = [("patch_128x256", 2, 112, 112, 64, 256, 3), ("patch_64x64", 1, 28, 28, 512, 256, 3), ("patch_128x64", 1, 56, 56, 64, 512, 3), ("tile_128x128", 2, 70, 70, 320, 256, 1)]
    specs = []
    for form, n, h, w, c, k, win in residual + pooled:
        g = GraphBuilder(form, dtype, n, h, w, c)
        if len(specs) < len(residual):
            g.conv(0, k, win, 1, win // 2, act="relu", bn=True, res=g.conv(0, k, win, 1, win // 2, act="none", bn=True))
        else:
            g.maxpool(g.conv(0, k, win, 1, win // 2, act="relu", bn=True), 2, 2, 0)
        specs.append(g.done())
    g = GraphBuilder("pair", dtype, 2, 28, 28, 64)
    g.dwconv(g.conv(0, 384, 1, 1, 0, act="relu6", bn=True), 3, 1, 1, act="relu6", bn=True)
    specs.append(g.done())
    fused = B.MT_SCHED_FUSE_POOL | B.MT_SCHED_FUSE_EXPAND
    for group in (specs[:len(residual)] + specs[-1:], specs[len(residual):]):
        mix = Mix(group, seed=47)
        try:
            ctx = mix.ctx
            print("case", dtype, [s.name for s in group], flush=True)
            for t, spec in enumerate(group[:-1]):
                assert ctx.op_form(t, 0).name.decode() == spec.name
            plain, tm = mix.run(ctx.sequential())
            assert tm["n_fused"] == 0
            convs = sum(op.kind == "conv" for spec in group[:-1] for op in spec.ops)
            for flags, n_fused in ((0, 0), (fused, 1 + sum(op.kind == "maxpool" for spec in group for op in spec.ops))):
                shared = ctx.schedule([[] for _ in group], 1, cu_share=[32] * len(group), flags=flags)
                for _ in range(2):
                    got, tm = mix.run(shared)
                    assert tm["n_fused"] == n_fused and shared.launch_forms()[0] >= convs
                    for p, q in zip(plain, got):
                        assert np.isfinite(p).all()
                        np.testing.assert_array_equal(p, q)
        finally:
            mix.close()
