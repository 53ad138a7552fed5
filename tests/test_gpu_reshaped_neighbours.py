"""Layers that read the result before them as a map of other channels (as many values in another shape), at places where a layer that reads it as it is shares a launch
with the one that forms it: against the oracle, which runs them one by one."""
import pytest

from tests.test_gpu_stage import run_stage_case
from workloads.configs import affine, conv, linear

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
