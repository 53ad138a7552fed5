"""Both table gradients of small tables in one launch: token counts around the four waves of a workgroup, row counts around the 64 and 256 that a wave scans
at a time, tokens with more rows than its list holds, features around a wave's 64, one sample and many; and larger tables on the kernels that
they stay on, with tokens of more rows than those keep in a list."""
import pytest

from tests.test_gpu_stage import run_stage_case
from workloads.configs import embedding, linear

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("vocab,s,d,micro,N", [(1, 1, 8, 1, 1), (2, 65, 64, 1, 1), (3, 64, 72, 2, 2), (4, 257, 64, 1, 1), (5, 85, 200, 3, 1), (7, 63, 64, 1, 4), (96, 32, 64, 2, 4),
                                               (500, 40, 8, 3, 2), (2000, 64, 64, 4, 2),
                                               (65, 512, 32, 8, 4),   # (16384 rows: beyond the line, 250 to a token)
                                               (100000, 3, 8, 1, 2), (100001, 3, 8, 1, 2)])   # (few rows, on both sides of the line for tables)
def test_embedding(vocab, s, d, micro, N, dtype):
    run_stage_case([embedding(vocab, s, d), linear(d, 16, False, rows=s)], dtype, micro, N, seed=vocab + s)
