"""Layer normalisation with the row in registers and beyond, in both types: one chunk of 8 features, a lane's second chunk begun and full, widths
that are no whole chunk, rows of more than 1024, row counts around the four of a workgroup and the slabs of the gradient."""
import pytest

from tests.test_gpu_stage import run_stage_case
from workloads.configs import layernorm, linear

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d,s,micro,N", [(8, 1, 1, 1), (8, 3, 3, 2), (64, 32, 2, 2), (72, 5, 1, 3), (504, 7, 2, 2), (512, 16, 1, 2), (520, 3, 3, 2), (1024, 2, 2, 2),
                                         (1016, 4, 1, 1), (1032, 3, 2, 2), (12, 5, 2, 2), (2048, 2, 1, 2), (16, 1024, 1, 2), (8, 4100, 1, 1)])
def test_layernorm(dtype, d, s, micro, N):
    run_stage_case([layernorm(d, s), linear(d, 24, False, rows=s)], dtype, micro, N, seed=d + s)
