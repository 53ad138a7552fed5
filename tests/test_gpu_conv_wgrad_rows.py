"""Weight gradients of 3 x 3 convolutions on runs of rows: one chunk of 128 positions, fewer, one more, and numbers of chunks on both sides of the
three that are staged; one slice and several, the last one shorter; maps of one row and of one column, tiles over many
images, the widest map whose run fits LDS and one wider; several tiles of either channels."""
import ctypes as C

import pytest

from paper_2410_14312_amd import load_library
from tests import routes
from tests.test_gpu_stage import run_stage_case
from workloads.configs import conv

CASES = [
    # (h, w, cin, cout, micro, N)
    (2, 2, 512, 512, 31, 1),     # 124 positions
    (4, 4, 512, 512, 8, 1),      # 128
    (3, 43, 512, 512, 1, 1),     # 129
    (2, 2, 64, 64, 300, 1),      # ten slices of one chunk
    (2, 2, 512, 512, 64, 1),     # two chunks
    (7, 7, 512, 512, 4, 2),      # four, the last one hardly begun
    (8, 8, 64, 192, 30, 1),      # slices
    (1, 61, 128, 128, 33, 1),
    (61, 1, 128, 128, 33, 1),
    (2, 75, 64, 128, 40, 1),
    (2, 76, 64, 128, 40, 1),
    (16, 16, 128, 64, 13, 2),
]


@pytest.mark.gpu
@pytest.mark.parametrize("h,w,cin,cout,micro,N", CASES)
def test_conv_wgrad_rows(h, w, cin, cout, micro, N):
    run_stage_case([conv(h, w, 64, cin, 1, 1, 0, True), conv(h, w, cin, cout, 3, 1, 1, False)], "bf16", micro, N, seed=h + 7 * w + cout)


class _Plan(C.Structure):
    _fields_ = [("slices", C.c_int), ("per_slice", C.c_int)]


@pytest.mark.parametrize("h,w,cin,cout,samples,slices", [(7, 7, 512, 512, 8, 1), (2, 2, 64, 64, 300, 10), (8, 8, 64, 192, 30, 8), (2, 75, 64, 128, 40, 16),
                                                         (2, 76, 64, 128, 40, 0), (16, 16, 128, 64, 26, 18), (16, 16, 128, 72, 26, 0)])
def test_slices_of_the_cases(h, w, cin, cout, samples, slices):
    plan = getattr(load_library(), "_ZN4tmps20conv_wgrad_rows_planERKNS_9ConvShapeEd")
    plan.restype, plan.argtypes = _Plan, [C.POINTER(routes._Conv), C.c_double]
    got = plan(C.byref(routes._Conv(samples, h, w, cin, h, w, cout, 3, 3, 1, 1)), 10.0)   # (the other kernels estimated at 10 us)
    assert got.slices == slices
    if slices:
        assert got.per_slice % 128 == 0 and (slices - 1) * got.per_slice < samples * h * w <= slices * got.per_slice
