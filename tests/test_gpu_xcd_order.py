"""How the 8 XCDs share the tiles of a contraction: as rectangles of 4 x 2 and 2 x 4 where both sides divide so, in strips elsewhere; on each kernel that
numbers its tiles so, with ragged last tiles, and on the kernel of asynchronous copies with the k-tiles' remainders by its five stages."""
import pytest

from tests import routes
from tests.test_gpu_stage import run_stage_case
from workloads.configs import linear

CASES = [   # rows, din, dout, kernel of the forward pass
    (1000, 3080, 512, "by_k"), (500, 3080, 760, "by_k"), (512, 3080, 776, "by_k"),
    (1000, 776, 512, "tiled"), (500, 776, 760, "tiled"), (1000, 72, 2000, "tiled"), (1030, 776, 256, "tiled"),
    (1000, 776, 3072, "async"), (1030, 776, 2000, "async"),
    (896, 512, 4096, "async"), (1024, 640, 3072, "async"), (896, 696, 2560, "async"), (1024, 768, 2560, "async"), (1024, 840, 3072, "async"),   # 8, 10, 11, 12, 14 k-tiles: every remainder
]


@pytest.mark.parametrize("rows,din,dout,kernel", CASES)
def test_routes(rows, din, dout, kernel):
    assert routes.dense_routes(linear(din, dout, False), "bf16", rows, 1)[0] == kernel


@pytest.mark.gpu
@pytest.mark.parametrize("rows,din,dout", [c[:3] for c in CASES])
def test_against_the_oracle(rows, din, dout):
    run_stage_case([linear(din, dout, False)], "bf16", rows, 1, seed=rows + din)
