"""Contractions at the edges of their kernels' ranges: the small kernel (16 x 16 to 32 x 32 outputs, the k range
shared by the waves; most of these layers' gradients are one launch of it) at its tile, step and wave-count borders, matrices whose rows are not whole 16-byte chunks (ragged loaders) or less
than one (gathering loaders), convolutions over channel counts that are not whole chunks, and the tiled fp32 kernel
with and without k-slices.  Against the oracle, all three passes, in both types."""
import pytest

from tests.test_gpu_stage import run_stage_case
from workloads.configs import conv, linear

pytestmark = pytest.mark.gpu

DENSE = [
    # (din, dout, micro, N)
    (3, 5, 2, 2),          # rows of less than a chunk: gathered
    (8, 4, 1, 1),          # one row
    (16, 33, 33, 1),       # half a step of k (bf16) / one (fp32), a tile and a column over
    (17, 31, 16, 2),       # a tail of one k
    (127, 129, 31, 2),     # 4 waves, tails in every pass
    (513, 65, 47, 1),      # 8 waves and a tail
    (1000, 10, 235, 1),    # a narrow output layer
    (72, 2601, 40, 2),     # odd output: ragged rows of dY in both gradients
    (1001, 1003, 300, 1),  # ragged everywhere, tiled
    (1001, 1003, 375, 4),  # the same with gradients in launches of their own
    (264, 520, 700, 1),    # fp32 tiles of several sizes, ragged last tiles
    (2048, 96, 512, 1),    # few tiles, long k: k-slices
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("din,dout,micro,N", DENSE)
def test_dense_edges(dtype, din, dout, micro, N):
    run_stage_case([linear(din, dout, False)], dtype, micro, N, seed=din + 3 * dout)


CONV = [
    # (h, w, cin, cout, r, stride, pad, micro, N)
    (9, 7, 3, 5, 3, 1, 1, 2, 2),     # neither channel count a chunk
    (8, 8, 6, 16, 3, 2, 1, 2, 2),    # stride 2, input channels no chunk (of 8)
    (8, 8, 16, 10, 1, 1, 0, 2, 2),   # 1x1: a dense layer with ragged output rows
    (12, 12, 4, 12, 3, 2, 1, 3, 1),  # whole chunks in fp32 only
    (16, 16, 8, 8, 5, 2, 2, 2, 1),   # 5x5 over parity classes
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("h,w,cin,cout,r,stride,pad,micro,N", CONV)
def test_conv_edges(dtype, h, w, cin, cout, r, stride, pad, micro, N):
    run_stage_case([conv(h, w, cin, cout, r, stride, pad, False)], dtype, micro, N, seed=h + cin * cout)


# Outputs of few 64 x 64 tiles over a long k (whole and partial k-tiles, ragged last tiles, a convolution's loaders in all
# passes).  tests/test_gpu_contraction_routes.py holds the kernel whose waves share k to sizes that are known to reach it.
BY_K = [
    [linear(1544, 584, False)],           # a tail of 8 in the forward pass, whole tiles in the weight gradient
    [linear(776, 1160, False)],
    [linear(2048, 512, False)],
]
BY_K_CONV = [
    [conv(8, 8, 256, 136, 3, 1, 1, False)],
    [conv(7, 7, 128, 264, 3, 2, 1, False)],
    [conv(14, 14, 512, 128, 1, 1, 0, False)],
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("micro,layers", [(330, l) for l in BY_K] + [(m, l) for l in BY_K_CONV for m in (5, 16)])
def test_few_tiles_long_k(dtype, micro, layers):
    run_stage_case(layers, dtype, micro, 1, seed=micro)


# Outputs of some 100 to 250 tiles of 128 x 128 (ragged last tiles, an odd number of k-tiles, a k tail, row sums over many
# column tiles).  tests/test_gpu_contraction_routes.py holds the kernel with asynchronous copies to sizes that reach it.
@pytest.mark.parametrize("layers,micro,N", [
    ([linear(776, 2312, False)], 500, 2),
    ([linear(1160, 1544, False)], 1030, 1),
    ([linear(64, 3080, False)], 520, 1),
    ([conv(30, 30, 64, 264, 3, 2, 1, False)], 10, 2),
    ([conv(15, 15, 72, 520, 3, 1, 1, False)], 24, 1),
])
def test_tiles_of_128(layers, micro, N):
    run_stage_case(layers, "bf16", micro, N, seed=micro)
