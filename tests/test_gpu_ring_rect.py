"""Rings on rectangles of 16 pixels (3x3 windows, stride 1, padding 1: the input pixels of a chunk of channels are copied once and the filters are packed in
operand order): both rectangles, ragged edges, several images, waves without a chunk and with two and three, against a plain
convolution on the CPU; the pooled epilogue against separate launches."""
import numpy as np
import pytest
import torch

from synth import GraphBuilder
from oracle import forward as OF
from oracle import ops as oops
from gpu_harness import Mix, assert_close
from paper_2111_14255_amd import api, binding as B
from test_gpu_ring import conv_ref

pytestmark = pytest.mark.gpu

CASES = [
    # rows and columns of the rectangle, n, h, w, channels of the 16-bit types (fp32: a half), output channels
    ("4x4_one_chunk", 1, 8, 8, 32, 40),
    ("4x4_ragged_rows_and_columns", 1, 7, 7, 64, 40),
    ("4x4_three_chunks_three_images", 3, 12, 12, 96, 72),
    ("2x8_ragged_columns", 1, 14, 14, 256, 264),
    ("2x8_nine_chunks", 1, 6, 8, 288, 96),
    ("4x4_seventeen_chunks", 1, 8, 4, 544, 48),
    ("4x4_nineteen_chunks_many_channels", 1, 7, 7, 608, 392),
    ("2x8_two_images_of_one_row", 2, 2, 8, 128, 264),
    ("4x4_larger_map", 1, 28, 28, 128, 136),
]


def rectangles(spec):
    m = api.Model(spec)
    try:
        return [m.op_rectangle(i) for i, op in enumerate(spec.ops) if op.kind == "conv"]
    finally:
        m.close()


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("name,n,h,w,c,k", CASES, ids=[c[0] for c in CASES])
def test_rectangles(name, n, h, w, c, k, dtype):
    c = c // 2 if dtype == "f32" else c
    g = GraphBuilder("t", dtype, n, h, w, c)
    a = g.conv(0, k, 3, 1, 1, act="relu", bn=True)
    d = g.new_tensor()                                   # the same with a residual, written at a channel offset
    g.conv(0, k, 3, 1, 1, act="relu6", bn=True, res=a, dst=d, c_off=4, c_tot=k + 4)
    g.conv(0, 4, 3, 1, 1, act="none", dst=d, c_off=0, c_tot=k + 4)
    spec = g.done()
    print("case", name, dtype, flush=True)
    mix = Mix([spec], seed=53)
    try:
        assert rectangles(spec)[:2] == [int(name[2])] * 2
        x = oops.round_array(mix.x[0], dtype)
        p = OF.prepare_params(spec, mix.raw[0])
        t0 = oops.round_array(torch.relu(conv_ref(x, p[0], 1, 1, 1)).float().contiguous().numpy(), dtype)
        t1 = (conv_ref(x, p[1], 1, 1, 1) + torch.from_numpy(t0).double()).clamp(0, 6)
        ref = torch.cat([conv_ref(x, p[2], 1, 1, 1), t1], dim=3).float().numpy()
        got, _ = mix.run(mix.ctx.sequential())
        assert_close(mix.ctx.read_tensor(0, a, t0.shape).astype(np.float32), t0, dtype, name)
        assert_close(got[0], ref.reshape(n, -1), dtype, name)
    finally:
        mix.close()


@pytest.mark.parametrize("n,h,w,c,k,columns", [(1, 8, 8, 64, 40, 4), (3, 12, 12, 96, 72, 4), (1, 6, 8, 288, 96, 8), (1, 14, 14, 512, 136, 8), (2, 2, 8, 128, 264, 8)])
def test_rectangles_pooled(n, h, w, c, k, columns):
    g = GraphBuilder("t", "f16", n, h, w, c)
    a = g.conv(0, k, 3, 1, 1, act="relu", bn=True)
    pl = g.maxpool(a, 2, 2, 0)
    g.gap(pl)
    print("case pooled", n, h, w, c, k, flush=True)
    spec = g.done()
    assert rectangles(spec)[0] == columns
    mix = Mix([spec], seed=54)
    try:
        shape = (n, h // 2, w // 2, k)
        _, tm = mix.run(mix.ctx.sequential(flags=B.MT_SCHED_FUSE_POOL))
        assert tm["n_fused"] == 1
        fused = mix.ctx.read_tensor(0, pl, shape)
        mix.run(mix.ctx.sequential())
        np.testing.assert_array_equal(fused.view(np.uint32), mix.ctx.read_tensor(0, pl, shape).view(np.uint32))
    finally:
        mix.close()
