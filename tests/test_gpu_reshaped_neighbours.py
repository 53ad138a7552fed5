"""Layers that read the result before them as a map of other channels (as many values in another shape), at places where a layer that reads it as it is shares a launch
with the one that forms it: against the oracle, which runs them one by one."""
import pytest

from tests.test_gpu_stage import run_stage_case
from workloads.configs import affine, bottleneck, conv, linear, maxpool

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("r", [1, 3])
@pytest.mark.parametrize("h,cout,c", [(8, 16, 4), (8, 16, 64), (32, 64, 16), (32, 64, 256), (32, 128, 32)])
def test_affine_behind_a_convolution(dtype, r, h, cout, c):
    """Forward the affine layer is the convolution's epilogue, and both layers' gradients are one pass (1 x 1 filters, 1024 positions and more): over its channels."""
    side = int((h * h * cout // c) ** 0.5)
    specs = [conv(h, h, 8, 64, 3, 1, 1, True), conv(h, h, 64, cout, r, 1, r // 2, False), affine(side, side, c, True), linear(h * h * cout, 8, False)]
    if side * side * c != h * h * cout:   # (a map that is no square)
        specs[2] = affine(h * h * cout // c // h, h, c, True)
    run_stage_case(specs, dtype, 2, 2, seed=h + c + r)


@pytest.mark.parametrize("h,cin,first,second", [(64, 256, 64, 64), (32, 64, 64, 64), (64, 64, 64, 16), (64, 128, 64, 64)])
def test_convolution_behind_a_join(h, cin, first, second):
    """The next block's first convolution leaves the join's launch (64 x 64 positions from 64 channels to 256) where it reads the join's 256 channels; the others
    here read it as maps of 64 and 128, one of them 64 x 64 again."""
    side = {(64, 256): (64, 64), (32, 64): (64, 64), (64, 64): (128, 128), (64, 128): (64, 128)}[h, cin]
    block, _, _ = bottleneck(h, 64, 64, 1, True)
    conv_ = conv(h, h, cin, first, 1, 1, 0, False)
    conv_.update(h=side[0], w=side[1])
    n = side[0] * side[1] * first // second
    run_stage_case([conv(h, h, 8, 64, 3, 1, 1, True)] + block + [conv_, affine(side[0], n // side[0], second, True), conv(side[0], n // side[0], second, 8, 1, 1, 0, False)],
                   "bf16", 4 if h == 32 else 1, 2, seed=h + cin + second, deep=True)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("h,w,c", [(8, 8, 16), (16, 4, 16), (4, 4, 64), (16, 16, 4), (8, 4, 32)])
def test_pooling_behind_an_affine_layer(dtype, h, w, c):
    """The pooling's input gradient and the affine layer's are one pass over the channels of both."""
    ho, wo = (h - 1) // 2 + 1, (w - 1) // 2 + 1
    run_stage_case([conv(8, 8, 8, 16, 3, 1, 1, False), affine(8, 8, 16, True), maxpool(h, w, c, k=3, stride=2, pad=1), linear(ho * wo * c, 8, False)], dtype, 3, 2,
                   seed=h + c, has_pool=True)
