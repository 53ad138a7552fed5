"""Attention's forward pass on both sides of the lines between its kernels: one block of 32 keys, 64 positions (two waves per workgroup), as
many tiles of 64 queries as send a launch to the tiled kernel (256 in bf16, 512 in fp32 and behind 1024 positions) and one fewer, with
numbers of (batch, head) pairs off a multiple of eight.  Against the oracle, both types."""
import pytest

from tests.test_gpu_stage import run_stage_case
from workloads.configs import attention, linear

pytestmark = pytest.mark.gpu

CASES = [
    # (s, d, heads, micro)
    (32, 64, 2, 5),
    (64, 64, 2, 128),     # 256 tiles of two waves
    (65, 128, 2, 64),     # 256 tiles, the last one's second block empty
    (161, 64, 1, 85),     # 255
    (129, 64, 2, 86),     # 516, a workgroup for one row
    (320, 64, 1, 52),
    (1025, 32, 1, 16),    # 272 behind 1024 positions
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("s,d,heads,micro", CASES)
def test_attention_forward(dtype, s, d, heads, micro):
    run_stage_case([linear(d, 3 * d, False, rows=s), attention(s, d, heads)], dtype, micro, 1, seed=s + d + heads)
