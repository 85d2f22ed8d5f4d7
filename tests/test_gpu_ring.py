"""The ring forms of the tile kernels (the waves of a workgroup deal the reduction out between them) and the fp32 tiles:
ragged pixel, channel and reduction counts, residual, channel offsets, groups and
the pooled epilogue, against a plain convolution on the CPU."""
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
    # name, n, h, w, c, k, window, stride, pad, groups, form of the 16-bit types and of fp32 (a ring's with its waves)
    ("16x16_tap_full_rings", 1, 14, 14, 256, 256, 3, 1, 1, 1, "ring_16x16/8", "ring_16x16/8"),
    ("16x16_tap_ragged_pixels_span_images", 3, 9, 7, 128, 72, 3, 1, 1, 1, "ring_16x16/8", "ring_16x16/4"),
    ("16x16_point_ragged", 1, 15, 13, 1024, 264, 1, 1, 0, 1, "ring_16x16/8", "ring_16x16/8"),
    ("16x16_chunk_c72", 1, 13, 13, 72, 200, 3, 1, 1, 1, "ring_16x16/4", "ring_16x16/8"),
    ("16x16_chunk_c200_unaligned_channels", 1, 10, 10, 200, 67, 3, 1, 1, 1, "ring_16x16/8", "ring_16x16/8"),
    ("216_rows", 1, 5, 5, 1536, 512, 3, 1, 1, 1, "tile_64x16", "ring_16x16/8"),
    ("16x16_1x7", 1, 17, 17, 192, 192, (1, 7), 1, (0, 3), 1, "ring_16x16/8", "ring_16x16/4"),
    ("16x16_stride2", 1, 28, 28, 256, 264, 3, 2, 1, 1, "ring_16x16/8", "ring_16x16/8"),
    ("32x16_tap_ragged", 1, 29, 27, 128, 136, 3, 1, 1, 1, "ring_32x16/4", "ring_32x16/4"),
    ("32x16_many_rows", 1, 14, 14, 512, 512, 3, 1, 1, 1, "ring_32x16/4", "ring_32x16/4"),
    ("four_waves_point", 1, 7, 7, 960, 160, 1, 1, 0, 1, "ring_16x16/4", "ring_16x16/8"),
    ("four_waves_uneven_rows_c264", 1, 4, 4, 264, 40, 1, 1, 0, 1, "ring_16x16/4", "ring_16x16/4"),
    ("four_waves_short_reduction", 1, 17, 17, 64, 100, 3, 1, 1, 1, "ring_16x16/4", "ring_16x16/4"),
    ("wide_map", 2, 60, 61, 64, 136, 3, 1, 1, 1, "patch_128x64", "tile_64x32"),
    ("chunk_c40", 2, 41, 40, 40, 132, 3, 1, 1, 1, "tile_64x64", "tile_64x64"),
    ("groups_of_96", 2, 13, 13, 192, 128, 3, 1, 1, 2, "ring_16x16/8", "ring_16x16/4"),
    ("channels_of_one_output_tile", 1, 6, 6, 512, 12, 3, 1, 1, 1, "ring_16x16/8", "registers_16x16"),
]
ACT = {"relu": torch.relu, "relu6": lambda v: v.clamp(0, 6), "none": lambda v: v}


def conv_ref(x, p, stride, pad, groups):
    w = torch.from_numpy(np.ascontiguousarray(p[0])).permute(0, 3, 1, 2).double()
    y = F.conv2d(torch.from_numpy(np.ascontiguousarray(x)).permute(0, 3, 1, 2).double(), w, torch.from_numpy(p[1]).double(), stride, pad, 1, groups)
    return y.permute(0, 2, 3, 1)


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("name,n,h,w,c,k,win,stride,pad,groups,form16,form32", CASES, ids=[c[0] for c in CASES])
def test_ring_and_fp32_tiles(name, n, h, w, c, k, win, stride, pad, groups, form16, form32, dtype):
    g = GraphBuilder("t", dtype, n, h, w, c)
    a = g.conv(0, k, win, stride, pad, act="relu6", bn=True, groups=groups)
    d = g.new_tensor()                                   # the same convolution with a residual, written at a channel offset
    off = 8 if k % 8 == 0 else 3
    g.conv(0, k, win, stride, pad, act="relu", bn=True, res=a, dst=d, c_off=off, c_tot=k + off, groups=groups)
    g.conv(0, off, win, stride, pad, act="none", dst=d, c_off=0, c_tot=k + off)
    spec = g.done()
    print("case", name, dtype, flush=True)
    mix = Mix([spec], seed=47)
    try:
        form = mix.ctx.op_form(0, 0)
        assert form.name.decode() + ("/%d" % form.ring_waves if form.ring_waves else "") == (form32 if dtype == "f32" else form16)
        x = oops.round_array(mix.x[0], dtype)
        p = OF.prepare_params(spec, mix.raw[0])
        t0 = oops.round_array(ACT["relu6"](conv_ref(x, p[0], stride, pad, groups)).float().contiguous().numpy(), dtype)
        t1 = ACT["relu"](conv_ref(x, p[1], stride, pad, groups) + torch.from_numpy(t0).double())
        ref = torch.cat([conv_ref(x, p[2], stride, pad, 1), t1], dim=3).float().numpy()
        first = None
        for sched in (mix.ctx.sequential(), mix.ctx.all_concurrent()):
            got, _ = mix.run(sched)
            assert_close(mix.ctx.read_tensor(0, a, t0.shape).astype(np.float32), t0, dtype, name)
            assert_close(got[0], ref.reshape(n, -1), dtype, name)
            first = got[0] if first is None else first
            assert np.array_equal(first.view(np.uint32), got[0].view(np.uint32))
    finally:
        mix.close()


@pytest.mark.parametrize("name,n,h,w,c,k", [("16x16", 1, 14, 14, 256, 256), ("32x16", 1, 28, 28, 128, 136), ("16x16_four_waves", 1, 12, 12, 64, 96)])
def test_pooled_epilogue_of_the_rings(name, n, h, w, c, k):
    g = GraphBuilder("t", "bf16", n, h, w, c)
    a = g.conv(0, k, 3, 1, 1, act="relu", bn=True)
    pl = g.maxpool(a, 2, 2, 0)
    g.gap(pl)
    print("case pooled", name, flush=True)
    mix = Mix([g.done()], seed=48)
    try:
        assert mix.ctx.op_form(0, 0).name.decode() == "ring_" + name[:5]
        shape = (n, h // 2, w // 2, k)
        _, tm = mix.run(mix.ctx.sequential(flags=B.MT_SCHED_FUSE_POOL))
        assert tm["n_fused"] == 1
        fused = mix.ctx.read_tensor(0, pl, shape)
        mix.run(mix.ctx.sequential())
        np.testing.assert_array_equal(fused.view(np.uint32), mix.ctx.read_tensor(0, pl, shape).view(np.uint32))
    finally:
        mix.close()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n,h,w,c,k,win,pad", [(2, 15, 17, 192, 100, 3, 1), (1, 29, 27, 128, 132, 3, 1), (1, 41, 39, 64, 92, 5, 2), (1, 60, 60, 512, 76, 1, 0),
                                               (1, 30, 31, 64, 4, 3, 1), (3, 40, 41, 64, 68, 3, 1)])
def test_residual_of_channels_in_fours(n, h, w, c, k, win, pad, dtype):
    """Channel counts and offsets that are multiples of 4 but not of 8 are stored, and the residual is read, in packs of four."""
    g = GraphBuilder("t", dtype, n, h, w, c)
    a = g.conv(0, k, win, 1, pad, act="none", bn=True)
    d = g.new_tensor()
    g.conv(0, k, win, 1, pad, act="relu", bn=True, res=a, dst=d, c_off=4, c_tot=k + 4)
    g.conv(0, 4, win, 1, pad, act="none", dst=d, c_off=0, c_tot=k + 4)
    spec = g.done()
    print("case", n, h, w, c, k, win, dtype, flush=True)
    mix = Mix([spec], seed=49)
    try:
        x = oops.round_array(mix.x[0], dtype)
        p = OF.prepare_params(spec, mix.raw[0])
        t0 = torch.from_numpy(oops.round_array(conv_ref(x, p[0], 1, pad, 1).float().contiguous().numpy(), dtype)).double()
        ref = torch.cat([conv_ref(x, p[2], 1, pad, 1), ACT["relu"](conv_ref(x, p[1], 1, pad, 1) + t0)], dim=3).float().numpy()
        got, _ = mix.run(mix.ctx.sequential())
        assert_close(got[0], ref.reshape(n, -1), dtype, "residual")
    finally:
        mix.close()
