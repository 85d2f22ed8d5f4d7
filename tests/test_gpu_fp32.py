"""fp32 convolution and fully connected layers on the matrix cores: every tiling, every way to gather an im2col row, ragged
channel and pixel counts, groups, residual and channel offsets, against the CPU oracle."""
import re

import pytest

from synth import GraphBuilder
from gpu_harness import Mix, assert_close

pytestmark = pytest.mark.gpu

CASES = [
    # name (the form the sizes lead to first), n, h, w, c, k, window, stride, pad, groups
    ("tile_32x32_uniform", 4, 57, 59, 64, 70, 3, 1, 1, 1),
    ("registers_32x32_elements_7x7", 2, 201, 190, 3, 64, 7, 2, 3, 1),
    ("tile_64x32_uniform", 1, 57, 55, 64, 100, 3, 1, 1, 1),
    ("tile_64x32_pieces_c20", 1, 60, 61, 20, 96, 3, 1, 1, 1),
    ("ring_32x16_uniform", 1, 29, 27, 128, 128, 3, 1, 1, 1),
    ("ring_16x16_uniform", 1, 7, 7, 96, 72, 3, 1, 1, 1),
    ("registers_16x16_pointwise_c144", 1, 14, 14, 144, 24, 1, 1, 0, 1),
    ("ring_16x16_pieces_c4_row_over_eight_taps", 3, 10, 11, 4, 9, 3, 1, 1, 1),
    ("ring_16x16_pieces_c12_stride2", 2, 15, 13, 12, 33, 5, 2, 2, 1),
    ("registers_16x16_elements_c3_11x11_stride4", 1, 59, 59, 3, 96, 11, 4, 0, 1),
    ("registers_64x64_elements_c1", 2, 9, 9, 1, 5, 3, 1, 1, 1),
    ("registers_16x16_elements_c33_asymmetric", 1, 9, 21, 33, 17, (1, 7), 1, (0, 3), 1),
    ("conv_direct_table_too_small_c255", 1, 6, 6, 255, 8, 3, 1, 1, 1),
    ("registers_16x16_groups_of_16", 2, 12, 12, 48, 96, 3, 1, 1, 3),
    ("ring_16x16_groups_of_4", 2, 12, 12, 8, 20, 3, 1, 1, 2),
    ("registers_16x16_groups_of_3", 1, 12, 12, 9, 12, 3, 1, 1, 3),
    ("tile_64x64_uniform", 4, 57, 57, 32, 70, 3, 1, 1, 1),
    ("tile_64x64_pieces_c20", 2, 57, 57, 20, 70, 3, 1, 1, 1),
    ("tile_64x16_uniform", 1, 41, 41, 32, 70, 3, 1, 1, 1),
    ("registers_32x32_uniform", 2, 57, 57, 16, 8, 3, 1, 1, 1),
    ("registers_32x32_pieces_c20", 2, 57, 57, 20, 8, 3, 1, 1, 1),
    ("registers_32x16_uniform", 1, 57, 57, 16, 24, 3, 1, 1, 1),
    ("registers_32x16_pieces_c20", 4, 28, 28, 20, 24, 3, 1, 1, 1),
    ("registers_32x16_elements_c3", 1, 29, 29, 3, 70, 3, 1, 1, 1),
    ("registers_16x16_pieces_c20", 1, 7, 7, 20, 8, 3, 1, 1, 1),
    ("registers_64x64_uniform_1x17", 8, 60, 60, 16, 64, (1, 17), 1, (0, 8), 1),
    ("registers_64x64_pieces_c12_17x1", 8, 60, 60, 12, 64, (17, 1), 1, (8, 0), 1),
    ("registers_32x32_pieces_c20_3x18", 2, 40, 40, 20, 70, (3, 18), 1, (1, 9), 1),
    ("gemv_one_pixel_one_channel", 1, 1, 1, 16, 1, 1, 1, 0, 1),
]


@pytest.mark.parametrize("name,n,h,w,c,k,win,stride,pad,groups", CASES, ids=[c[0] for c in CASES])
def test_fp32_convolution(name, n, h, w, c, k, win, stride, pad, groups):
    g = GraphBuilder("t", "f32", n, h, w, c)
    a = g.conv(0, k, win, stride, pad, act="none", bn=True, groups=groups)
    d = g.new_tensor()                                   # a second convolution with a residual, written at a channel offset
    g.conv(0, k, win, stride, pad, act="relu6", bn=True, groups=groups, res=a, dst=d, c_off=3, c_tot=k + 5)
    g.conv(0, 3, win, stride, pad, act="none", dst=d, c_off=0, c_tot=k + 5)
    g.conv(0, 2, win, stride, pad, act="relu", dst=d, c_off=k + 3, c_tot=k + 5)
    spec = g.done()
    print("case", name, flush=True)
    mix = Mix([spec], seed=41)
    try:
        assert mix.ctx.op_form(0, 0).name.decode() == re.match(r"(tile|ring|registers)_\d+x\d+|conv_direct|gemv", name).group(0)
        got, _ = mix.run(mix.ctx.sequential())
        assert_close(got[0], mix.oracle()[0], "f32", name)
    finally:
        mix.close()


@pytest.mark.parametrize("n,c,k", [(1, 512, 1000), (2, 100, 11), (8, 4096, 64), (9, 512, 70), (3, 10, 7), (40, 2050, 33)])
def test_fp32_fully_connected(n, c, k):
    g = GraphBuilder("t", "f32", n, 1, 1, c)
    g.fc(0, k, act="relu")
    print("case fc", n, c, k, flush=True)
    mix = Mix([g.done()], seed=42)
    try:
        got, _ = mix.run(mix.ctx.sequential())
        assert_close(got[0], mix.oracle()[0], "f32")
    finally:
        mix.close()
