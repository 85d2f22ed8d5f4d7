"""The patch kernels: filters are requested a number of steps ahead, across the chunks of 64 channels, and the last chunk requests none; one, two and
three to five chunks on every tile, channel counts that are a multiple of eight and that are not, against a convolution in 64 bits on the CPU."""
import numpy as np
import pytest

from synth import GraphBuilder
from oracle import forward as OF
from oracle import ops as oops
from gpu_harness import Mix, assert_close
from paper_2111_14255_amd import binding as B
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


# The widest tile: one group of waves up to four chunks of channels, two beyond
@pytest.mark.parametrize("c,k,split", [(256, 131, 1), (256, 136, 1), (320, 131, 1), (320, 136, 1), (384, 72, 3), (512, 72, 3)])
def test_widest_tile(c, k, split):
    n, h, w = 5, 44, 75
    g = GraphBuilder("t", "f16", n, h, w, c)
    a = g.conv(0, k, 3, 1, 1, act="relu", bn=True)
    b = g.conv(0, k, 3, 1, 1, act="relu6", bn=True, res=a)
    g.gap(b)
    spec = g.done()
    print("case widest", c, k, split, flush=True)
    mix = Mix([spec], seed=67)
    try:
        for op in (0, 1):
            assert mix.ctx.op_form(0, op).name.decode() == "patch_128x256" and mix.ctx.op_form(0, op).split_k == split
        x = oops.round_array(mix.x[0], "f16")
        p = OF.prepare_params(spec, mix.raw[0])
        t0 = oops.round_array(conv_ref(x, p[0], 1, 1, 1).clamp(min=0).float().numpy(), "f16")
        t1 = (conv_ref(x, p[1], 1, 1, 1).numpy() + t0).clip(0, 6)
        mix.run(mix.ctx.sequential())
        assert_close(mix.ctx.read_tensor(0, a, t0.shape).astype(np.float32), t0, "f16", "widest")
        assert_close(mix.ctx.read_tensor(0, b, t1.shape).astype(np.float32), oops.round_array(t1.astype(np.float32), "f16"), "f16", "widest, residual")
    finally:
        mix.close()


@pytest.mark.parametrize("n,h,w,c,k", [(5, 82, 82, 128, 72), (5, 44, 76, 256, 136), (5, 44, 76, 320, 136)])
def test_widest_tile_pooled(n, h, w, c, k):
    g = GraphBuilder("t", "f16", n, h, w, c)
    a = g.conv(0, k, 3, 1, 1, act="relu", bn=True)
    pl = g.maxpool(a, 2, 2, 0)
    g.gap(pl)
    print("case widest pooled", n, h, w, c, k, flush=True)
    mix = Mix([g.done()], seed=68)
    try:
        assert mix.ctx.op_form(0, 0).name.decode() == "patch_128x256"
        shape = (n, h // 2, w // 2, k)
        _, tm = mix.run(mix.ctx.sequential(flags=B.MT_SCHED_FUSE_POOL))
        assert tm["n_fused"] == 1
        fused = mix.ctx.read_tensor(0, pl, shape)
        mix.run(mix.ctx.sequential())
        np.testing.assert_array_equal(fused.view(np.uint32), mix.ctx.read_tensor(0, pl, shape).view(np.uint32))
    finally:
        mix.close()


def test_widest_tile_walks_with_the_same_bits():
    """Launches cut to a share of the units have both numbers of groups in one kernel."""
    specs = []
    for h, w, c, k in [(44, 75, 256, 136), (44, 75, 320, 136), (44, 75, 512, 72), (82, 82, 128, 72)] * 2:
        g = GraphBuilder("t%d" % c, "f16", 5, h, w, c)
        g.gap(g.conv(0, k, 3, 1, 1, act="relu", bn=True))
        specs.append(g.done())
    print("case widest walking", flush=True)
    mix = Mix(specs, seed=69)
    try:
        assert all(mix.ctx.op_form(t, 0).name.decode() == "patch_128x256" for t in range(len(specs)))
        plain, _ = mix.run(mix.ctx.sequential())
        shared = mix.ctx.schedule([[] for _ in specs], 1, cu_share=[32] * len(specs))
        for _ in range(2):
            got, _ = mix.run(shared)
            assert shared.launch_forms()[0] >= len(specs)
            for p, q in zip(plain, got):
                assert np.isfinite(p).all()
                np.testing.assert_array_equal(p, q)
    finally:
        mix.close()
