"""Input gradients of strided 1 x 1 convolutions that other layers' contributions precede: added in place at the positions that the filter reaches.  Maps
that the stride divides and not, one position, strides of two and three; behind a ReLU, behind a layer without activation (nothing to mask) and at the stage
input; as the only reader, where the whole map is written as before, and behind a block with an identity join."""
import pytest

from tests.test_gpu_stage import run_stage_case
from workloads.configs import affine, avgpool, bottleneck, conv, linear, resadd, softmax_ce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("h,cin,width", [(8, 16, 16), (9, 32, 8), (1, 8, 8), (16, 64, 40), (7, 24, 64)])
@pytest.mark.parametrize("below", ["relu", "none", "input"])
def test_projection_blocks(h, cin, width, below, dtype):
    first = [] if below == "input" else [conv(h, h, 8, cin, 1, 1, 0, below == "relu")]
    block, ho, cout = bottleneck(h, cin, width, 2, True)
    run_stage_case(first + block + [avgpool(ho, ho, cout), linear(cout, 10, False), softmax_ce(10)], dtype, 3, 2, seed=h + cin)


def strided(h, cin, cout, stride, src):
    ho = (h - 1) // stride + 1
    return conv(h, h, cin, cout, 1, stride, 0, False, src=src), ho


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("h,stride", [(9, 3), (10, 3), (11, 2)])
def test_two_strided_readers(h, stride, dtype):
    """The second one read waits, the first one is written over the whole map."""
    one, ho = strided(h, 16, 24, stride, 1)
    two, _ = strided(h, 16, 24, stride, 3)
    run_stage_case([conv(h, h, 8, 16, 1, 1, 0, True), one, affine(ho, ho, 24, False), two, affine(ho, ho, 24, False), resadd(ho, ho, 24, src_b=3, relu=True)],
                   dtype, 2, 3, seed=h)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_alone(dtype):
    one, ho = strided(7, 16, 24, 2, 1)
    run_stage_case([conv(7, 7, 8, 16, 1, 1, 0, True), one, affine(ho, ho, 24, True)], dtype, 2, 2, seed=3)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_beside_a_join(dtype):
    """The strided layer reads the result of an identity block, and a 3 x 3 layer with a stride after it."""
    h, c = 6, 16
    block, _, _ = bottleneck(h, c, 4, 1, False)
    one, ho = strided(h, c, 24, 2, 1)
    two = conv(h, h, c, 24, 3, 2, 1, False, src=3)
    run_stage_case([conv(h, h, 8, c, 1, 1, 0, True)] + block + [one, affine(ho, ho, 24, False), two, affine(ho, ho, 24, False), resadd(ho, ho, 24, src_b=3, relu=True)],
                   dtype, 2, 2, seed=4)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("h,cin,width,stride", [(4, 64, 256, 2), (7, 40, 200, 2), (1, 8, 192, 2), (5, 24, 300, 3)])
def test_in_slices(h, cin, width, stride, dtype):
    """Few positions and a long contraction: its slices' sums are of the positions that the filter reaches."""
    from tests.routes import DENSE, _functions
    block, ho, cout = bottleneck(h, cin, width, stride, True)
    assert _functions()[0](6 * ho * ho, cin, cout, False, 2 if dtype == "bf16" else 4, DENSE).slices > 1
    run_stage_case([conv(h, h, 8, cin, 1, 1, 0, True)] + block + [avgpool(ho, ho, cout), linear(cout, 10, False), softmax_ce(10)], dtype, 3, 2, seed=h + cin)
