"""The tile kernels whose filters go straight to registers: a stage's filters take the place of those of the stage just multiplied, and the first stages are
requested together; one to seven stages, a half empty last one, groups, splits, and channel counts that are a multiple of eight and that are not,
against a convolution in 64 bits on the CPU."""
import numpy as np
import pytest

from synth import GraphBuilder
from oracle import forward as OF
from oracle import ops as oops
from gpu_harness import Mix, assert_close
from test_gpu_ring import conv_ref

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("name,slices,stages,split,n,h,w,c,k,win,pad,groups", [
    ("tile_128x64", 1, 1, 1, 5, 36, 48, 40, 72, 1, 0, 1), ("tile_128x64", 1, 2, 1, 8, 53, 20, 72, 72, 1, 0, 1), ("tile_128x64", 1, 3, 1, 8, 43, 26, 192, 67, 1, 0, 1),
    ("tile_128x64", 1, 4, 1, 8, 48, 23, 256, 72, 1, 0, 1), ("tile_128x64", 1, 5, 1, 5, 30, 56, 320, 72, 1, 0, 1), ("tile_128x64", 1, 6, 1, 8, 50, 21, 384, 67, 1, 0, 1),
    ("tile_128x64", 1, 2, 1, 5, 35, 49, 192, 136, 1, 0, 2),
    ("tile_64x64", 2, 1, 1, 8, 29, 20, 72, 67, 1, 0, 1), ("tile_64x64", 2, 2, 1, 3, 42, 33, 192, 67, 1, 0, 1), ("tile_64x64", 2, 3, 1, 3, 26, 54, 320, 67, 1, 0, 1),
    ("tile_64x64", 2, 4, 1, 5, 54, 17, 512, 72, 1, 0, 1), ("tile_64x64", 2, 5, 1, 5, 19, 44, 64, 72, 3, 1, 1), ("tile_64x64", 2, 6, 1, 3, 50, 29, 72, 67, 3, 1, 1),
    ("tile_64x64", 2, 7, 1, 3, 48, 60, 96, 40, 3, 1, 1), ("tile_64x64", 2, 4, 1, 5, 20, 32, 96, 260, 3, 1, 2), ("tile_64x64", 2, 18, 3, 1, 50, 43, 256, 67, 3, 1, 1),
    ("tile_64x64", 2, 23, 5, 5, 55, 10, 320, 40, 3, 1, 1)])
def test_packed_filters(name, slices, stages, split, n, h, w, c, k, win, pad, groups, dtype):
    g = GraphBuilder("t", dtype, n, h, w, c)
    a = g.conv(0, k, win, 1, pad, act="relu", bn=True, groups=groups)
    g.gap(a)
    spec = g.done()
    print("case", name, stages, split, n, h, w, c, k, win, groups, dtype, flush=True)
    mix = Mix([spec], seed=63)
    try:
        f = mix.ctx.op_form(0, 0)
        assert (f.name.decode(), f.stage_slices, f.split_k) == (name, slices, split) and -(-win * win * c // groups // (64 * slices)) == stages
        x = oops.round_array(mix.x[0], dtype)
        p = OF.prepare_params(spec, mix.raw[0])
        ref = conv_ref(x, p[0], 1, pad, groups).clamp(min=0).numpy()
        mix.run(mix.ctx.sequential())
        got = mix.ctx.read_tensor(0, a, ref.shape).astype(np.float32)
        assert_close(got, oops.round_array(ref.astype(np.float32), dtype), dtype, name)
    finally:
        mix.close()
