"""1x1 convolutions and classifiers keep a non-finite pixel to itself: the reduction is padded to whole stages of the tile kernels,
and what lies behind a pixel's channels in memory is the next pixel, the next image or the next group."""
import numpy as np
import pytest
import torch

from synth import GraphBuilder
from oracle import forward as OF
from oracle import ops as oops
from gpu_harness import Mix, TOL
from paper_2111_14255_amd import binding as B

pytestmark = pytest.mark.gpu

# n, h, w, c, k, groups: channels that are an odd number of 128-byte rows (64 elements of a 16-bit type, 32 of fp32), and one
# even number beside them, on maps from the narrow tiles (64 x 16) to the wide ones
SHAPES = {
    "f16": [(2, 20, 20, 64, 64, 1), (2, 60, 60, 64, 64, 1), (1, 56, 56, 64, 72, 1), (2, 9, 13, 192, 64, 1), (2, 60, 60, 192, 64, 1),
            (2, 60, 60, 192, 72, 1), (2, 28, 28, 320, 64, 1), (1, 56, 56, 320, 72, 1), (1, 56, 56, 320, 136, 1), (100, 1, 1, 192, 520, 1),
            (2, 28, 28, 384, 128, 2), (2, 20, 20, 128, 64, 1)],
    "f32": [(2, 28, 28, 32, 64, 1), (2, 28, 28, 32, 136, 1), (1, 56, 56, 96, 64, 1), (1, 56, 56, 96, 72, 1), (2, 28, 28, 96, 136, 1),
            (2, 60, 60, 288, 72, 1), (100, 1, 1, 96, 520, 1), (2, 28, 28, 192, 128, 2), (2, 28, 28, 64, 64, 1)],
}
SHAPES["bf16"] = SHAPES["f16"]
CASES = [(d,) + s for d in ("f16", "bf16", "f32") for s in SHAPES[d]]


@pytest.mark.parametrize("dtype,n,h,w,c,k,groups", CASES)
def test_pointwise_layers_keep_non_finite_pixels_to_themselves(dtype, n, h, w, c, k, groups):
    g = GraphBuilder("t", dtype, n, h, w, c)
    g.conv(0, k, 1, act="none", bn=False, groups=groups)
    spec = g.done()
    print("case", dtype, n, h, w, c, k, groups, flush=True)
    mix = Mix([spec], seed=53)
    try:
        x = mix.x[0]
        x[0, 0, 0, 0] = np.inf                               # channel 0 is the first one behind the pixel or group before
        x[0, h // 2, w // 2, 3] = np.nan
        x[n - 1, 0, 0, 5] = -np.inf                          # behind the last pixel of the image before, where there is one
        x[n - 1, h - 1, w - 1, c // groups * (groups - 1)] = np.nan      # first channel of the last group
        mix.inputs[0] = mix.ctx.make_input(0, x)
        got, _ = mix.run(mix.ctx.sequential())
        p = OF.prepare_params(spec, mix.raw[0])[0]
        wt = torch.from_numpy(np.ascontiguousarray(p[0])).reshape(groups, k // groups, c // groups).double()
        xs = torch.from_numpy(oops.round_array(x, dtype)).reshape(-1, groups, c // groups).double()
        ref = torch.cat([xs[:, i] @ wt[i].T for i in range(groups)], 1) + torch.from_numpy(p[1]).double()
        ref = ref.numpy().reshape(n, -1)
        bad = ~np.isfinite(ref)
        assert bad.any() and not bad.all()
        assert np.array_equal(~np.isfinite(got[0]), bad)
        assert float(np.abs(got[0][~bad] - ref[~bad]).max()) <= TOL[dtype] * float(np.abs(ref[~bad]).max())
    finally:
        mix.close()


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_fused_pair_has_the_bits_of_two_launches_beside_non_finite_pixels(dtype):
    g = GraphBuilder("blk", dtype, 1, 14, 14, 64)
    e = g.conv(0, 384, 1, act="none", bn=True)
    g.dwconv(e, 3, 1, 1, act="none", bn=True)
    mix = Mix([g.done()], seed=54)
    try:
        x = mix.x[0]
        x[0, 6, 6, 0] = np.nan
        x[0, 9, 0, 17] = np.inf
        mix.inputs[0] = mix.ctx.make_input(0, x)
        plain, tm = mix.run(mix.ctx.sequential())
        wide = mix.ctx.read_tensor(0, e, (1, 14, 14, 384))
        assert tm["n_fused"] == 0
        fused, tm = mix.run(mix.ctx.sequential(flags=B.MT_SCHED_FUSE_EXPAND))
        assert tm["n_fused"] == 1
        assert not np.isfinite(plain[0]).all() and np.isfinite(plain[0]).any()
        np.testing.assert_array_equal(plain[0], fused[0])
        np.testing.assert_array_equal(wide, mix.ctx.read_tensor(0, e, (1, 14, 14, 384)))
    finally:
        mix.close()
