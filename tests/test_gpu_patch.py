"""The patch kernels: filters are requested a number of steps ahead, across the chunks of 64 channels, and the last chunk requests none; one, two and
three to five chunks on every tile, channel counts that are a multiple of eight and that are not, against a convolution in 64 bits on the CPU."""
import numpy as np
import pytest

from synth import GraphBuilder
from oracle import forward as OF
from oracle import ops as oops
from gpu_harness import Mix, assert_close
from test_gpu_ring import conv_ref

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("name,n,h,w,c,k", [
    ("patch_64x32", 3, 90, 61, 64, 40), ("patch_64x32", 5, 66, 50, 128, 40), ("patch_64x32", 2, 41, 33, 256, 67), ("patch_64x32", 3, 18, 51, 320, 67),
    ("patch_64x64", 1, 79, 65, 64, 67), ("patch_64x64", 2, 40, 60, 128, 72), ("patch_64x64", 1, 79, 52, 192, 67), ("patch_64x64", 3, 26, 53, 320, 72),
    ("patch_128x64", 5, 27, 64, 64, 67), ("patch_128x64", 2, 74, 58, 128, 72), ("patch_128x64", 3, 45, 64, 192, 67), ("patch_128x64", 3, 83, 33, 256, 72),
    ("patch_128x128", 3, 38, 71, 64, 131), ("patch_128x128", 3, 73, 75, 128, 72), ("patch_128x128", 5, 77, 43, 192, 67),
    ("patch_128x256", 5, 82, 82, 64, 72), ("patch_128x256", 5, 88, 77, 128, 72), ("patch_128x256", 3, 73, 79, 192, 131)])
def test_patch_chunks(name, n, h, w, c, k, dtype):
    g = GraphBuilder("t", dtype, n, h, w, c)
    a = g.conv(0, k, 3, 1, 1, act="relu", bn=True)
    g.gap(a)
    spec = g.done()
    print("case", name, n, h, w, c, k, dtype, flush=True)
    mix = Mix([spec], seed=61)
    try:
        assert mix.ctx.op_form(0, 0).name.decode() == name and mix.ctx.op_form(0, 0).split_k == 1
        x = oops.round_array(mix.x[0], dtype)
        p = OF.prepare_params(spec, mix.raw[0])
        ref = conv_ref(x, p[0], 1, 1, 1).clamp(min=0).numpy()
        mix.run(mix.ctx.sequential())
        got = mix.ctx.read_tensor(0, a, ref.shape).astype(np.float32)
        assert_close(got, oops.round_array(ref.astype(np.float32), dtype), dtype, name)
    finally:
        mix.close()
