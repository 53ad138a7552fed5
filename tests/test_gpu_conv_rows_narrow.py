"""Convolutions on runs of rows in tiles of 32 columns: column tiles that are full, half and hardly full, row tiles that end inside an image, a
group of waves without a tap in the last step (9, 25 and 27 taps among four groups) and enough tiles to lie on both sides of the
line to wider ones."""
import pytest

from tests.test_gpu_stage import run_stage_case
from workloads.configs import conv

pytestmark = pytest.mark.gpu

CASES = [
    # (h, w, cin, cout, r, micro, N)
    (2, 2, 64, 64, 3, 1, 1),
    (2, 2, 128, 96, 3, 37, 1),
    (4, 4, 64, 8, 3, 5, 2),
    (3, 3, 192, 40, 3, 11, 1),
    (4, 5, 64, 72, 5, 7, 1),
    (2, 2, 512, 512, 3, 16, 2),
    (4, 4, 256, 512, 3, 64, 1),    # 256 tiles of 32 columns
    (4, 4, 256, 512, 3, 66, 1),    # more
]


@pytest.mark.parametrize("h,w,cin,cout,r,micro,N", CASES)
def test_conv_rows_narrow(h, w, cin, cout, r, micro, N):
    run_stage_case([conv(h, w, 64, cin, 1, 1, 0, True), conv(h, w, cin, cout, r, 1, r // 2, False)], "bf16", micro, N, seed=h + 7 * w + cout)
