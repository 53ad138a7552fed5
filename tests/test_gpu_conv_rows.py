"""Convolutions of unit stride that keep the map size, over whole 64-channel blocks, on the kernel that keeps a run of
input rows in LDS: tiles that start and end inside images, maps of one row or column, runs that reach before the first and past the
last position, one to three channel blocks, column tiles that are not full, 5 x 5 filters; on tiles of 32 columns and on each variant with wider ones
(tests/test_gpu_contraction_routes.py asks the library which a case runs on)."""
import pytest

from tests.test_gpu_stage import run_stage_case
from workloads.configs import conv

pytestmark = pytest.mark.gpu

CASES = [
    # (h, w, cin, cout, r, micro, N)
    (8, 8, 64, 64, 3, 4, 2),
    (7, 9, 64, 72, 3, 3, 2),
    (1, 13, 64, 64, 3, 5, 1),
    (13, 1, 64, 64, 3, 5, 1),
    (14, 14, 192, 64, 3, 3, 1),
    (2, 2, 128, 128, 3, 50, 2),
    (5, 7, 64, 128, 5, 4, 1),
    (16, 16, 64, 192, 3, 20, 2),
    (40, 40, 64, 64, 3, 9, 2),
]
# the same where there are more tiles, with the variants of the forward pass and of the input gradient (None: another kernel)
WIDE = [
    (4, 5, 128, 72, 5, 285, 1, 413, None),
    (5, 7, 64, 128, 5, 251, 1, 823, 413),
    (1, 13, 64, 136, 3, 506, 1, 422, None),
    (13, 1, 64, 128, 3, 642, 1, 422, 1413),
    (7, 9, 64, 200, 3, 285, 1, 443, None),
    (3, 5, 192, 72, 3, 727, 1, 823, None),
    (14, 14, 192, 64, 3, 132, 1, 823, 443),
]


@pytest.mark.parametrize("h,w,cin,cout,r,micro,N", CASES)
def test_conv_rows(h, w, cin, cout, r, micro, N):
    run_stage_case([conv(h, w, 64, cin, 1, 1, 0, True), conv(h, w, cin, cout, r, 1, r // 2, False)], "bf16", micro, N, seed=h + 7 * w + cout)


@pytest.mark.parametrize("h,w,cin,cout,r,micro,N,forward,input_gradient", WIDE)
def test_conv_rows_wide(h, w, cin, cout, r, micro, N, forward, input_gradient):
    run_stage_case([conv(h, w, 64, cin, 1, 1, 0, True), conv(h, w, cin, cout, r, 1, r // 2, False)], "bf16", micro, N, seed=h + 7 * w + cout)
