"""The matrix-vector kernel: eight channels of a pixel are stored at once where channel counts and offsets allow it and one by one elsewhere;
channel counts around a workgroup's eight and the bank's 64, one to eight pixels, residual and channel offset, against a plain product on the CPU."""
import numpy as np
import pytest
import torch

from synth import GraphBuilder
from oracle import forward as OF
from oracle import ops as oops
from gpu_harness import Mix, assert_close
from test_gpu_ring import conv_ref

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("n,c,k,off", [(1, 512, 1000, 8), (1, 64, 8, 8), (1, 136, 13, 8), (2, 264, 64, 3), (1, 72, 65, 0), (3, 512, 24, 16), (5, 64, 9, 1), (1, 4096, 7, 8)])
def test_matrix_vector(n, c, k, off, dtype):
    g = GraphBuilder("t", dtype, n, 1, 1, c)
    a = g.conv(0, k, 1, act="relu", bn=True)
    d = g.new_tensor()                                   # the same with a residual, written at a channel offset
    g.conv(0, k, 1, act="none", bn=True, res=a, dst=d, c_off=off, c_tot=k + off)
    if off:
        g.conv(0, off, 1, act="none", dst=d, c_off=0, c_tot=k + off)
    spec = g.done()
    print("case", n, c, k, off, dtype, flush=True)
    mix = Mix([spec], seed=59)
    try:
        assert mix.ctx.op_form(0, 0).name.decode() == "gemv"
        x = oops.round_array(mix.x[0], dtype)
        p = OF.prepare_params(spec, mix.raw[0])
        t0 = oops.round_array(torch.relu(conv_ref(x, p[0], 1, 0, 1)).float().contiguous().numpy(), dtype)
        t1 = conv_ref(x, p[1], 1, 0, 1) + torch.from_numpy(t0).double()
        ref = (torch.cat([conv_ref(x, p[2], 1, 0, 1), t1], dim=3) if off else t1).float().numpy()
        got, _ = mix.run(mix.ctx.sequential())
        assert_close(mix.ctx.read_tensor(0, a, t0.shape).astype(np.float32), t0, dtype, "matrix-vector")
        assert_close(got[0], ref.reshape(n, -1), dtype, "matrix-vector")
    finally:
        mix.close()
