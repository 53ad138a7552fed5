"""Attention at the edges of its kernels' ranges: 32 and 64 features per head on the MFMA path and other head sizes on the
generic one, sequences of one position, around the 32-row blocks and the LDS tiles (64 rows in bf16, 32 in fp32) and long
enough for the wider workgroups, few and many (batch, head) pairs.  Against the oracle, forward and backward, both types."""
import pytest

from tests.test_gpu_stage import run_stage_case
from workloads.configs import attention, linear

pytestmark = pytest.mark.gpu

CASES = [
    # (s, d, heads, micro, N)
    (1, 64, 2, 2, 2),
    (31, 64, 1, 2, 2),
    (33, 96, 3, 2, 1),
    (64, 128, 4, 1, 2),
    (97, 128, 2, 2, 2),
    (130, 192, 3, 2, 1),
    (70, 48, 3, 2, 2),      # 16 features per head: generic
    (40, 128, 1, 1, 2),     # 128 features per head: generic
    (200, 256, 4, 24, 1),   # enough (batch, head) pairs for the tiled forward kernel
    (65, 256, 8, 40, 1),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("s,d,heads,micro,N", CASES)
def test_attention_edges(dtype, s, d, heads, micro, N):
    run_stage_case([linear(d, 3 * d, False, rows=s), attention(s, d, heads)], dtype, micro, N, seed=s + d + heads)
