"""Attention's gradients, whose one launch holds workgroups for queries and for keys: numbers of (batch, head) pairs below, at and off a
multiple of eight, blocks that end at, before and behind the 128 rows of a workgroup and the 64 (bf16) or 32 (fp32) of a tile, and
launches on both sides of the line between two and four waves.  Against the oracle, both types."""
import pytest

from tests.test_gpu_stage import run_stage_case
from workloads.configs import attention, linear

pytestmark = pytest.mark.gpu

CASES = [
    # (s, d, heads, micro, N)
    (127, 32, 1, 1, 1),     # one pair, 32 features
    (128, 64, 1, 7, 1),     # seven pairs, 64 features
    (129, 96, 3, 3, 1),     # nine pairs
    (192, 64, 2, 4, 1),     # eight pairs, a workgroup half full
    (257, 128, 2, 3, 2),
    (160, 64, 1, 13, 1),    # thirteen pairs, a last tile half full
    (128, 128, 4, 31, 1),   # 124 pairs of 32 features: two waves
    (128, 128, 4, 32, 1),   # 128: four
    (32, 64, 2, 16, 1),
    (2, 128, 2, 9, 1),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("s,d,heads,micro,N", CASES)
def test_attention_backward(dtype, s, d, heads, micro, N):
    run_stage_case([linear(d, 3 * d, False, rows=s), attention(s, d, heads)], dtype, micro, N, seed=s + d + heads)
