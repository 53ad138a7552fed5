"""Contractions on the kernels that only some sizes reach: waves that share a tile by k ("by_k"), 128 x 128 tiles with
asynchronous copies ("async") and convolutions on runs of input rows kept in LDS ("rows", its five variants), each in the forward
pass, the input gradient and the weight gradient, with and without k-slices, ragged last tiles and k tails.  Which kernel a
case runs on is checked without a GPU by asking the library's planning functions (tests/routes.py), so that a change of the
rules cannot quietly empty these tests."""
import pytest

from tests import routes
from tests.test_gpu_conv_rows import CASES as CONV_ROWS_CASES, WIDE as CONV_ROWS_WIDE
from tests.test_gpu_stage import run_stage_case
from workloads.configs import conv, linear

DENSE = [
    # (dtype, rows, din, dout, (forward, input gradient, weight gradient); None: not of interest here)
    ("bf16", 760, 2056, 712, ("by_k", None, None)),            # a k tail of 8, ragged tiles
    ("bf16", 2112, 2672, 72, ("by_k split", None, None)),
    ("bf16", 609, 392, 1512, (None, "joint tiled", "joint tiled")),   # (see POINTWISE)
    ("bf16", 520, 224, 4192, (None, "joint small", "joint small")),
    ("bf16", 1217, 1200, 200, (None, "joint small", "joint small")),
    ("bf16", 4120, 1312, 80, (None, None, "by_k split")),
    ("f32", 201, 768, 2760, ("by_k", None, None)),
    ("f32", 141, 3856, 748, (None, "by_k", None)),
    ("f32", 753, 2704, 200, (None, None, "by_k")),
    ("f32", 236, 748, 1584, ("small", None, None)),
    ("f32", 262, 1552, 940, (None, "small", None)),
    ("bf16", 1000, 776, 2952, ("async", "by_k", "async")),     # 13 k-tiles, the last one short
    ("bf16", 1003, 2952, 776, ("by_k", "async", "async")),
    ("bf16", 3745, 3464, 72, (None, None, "async split")),
    ("bf16", 4096, 1024, 512, (None, "async", None)),            # outputs of 256 tiles of 128 x 128 ...
    ("bf16", 4096, 1024, 1024, ("async", "async", None)),
    ("bf16", 640, 1024, 5504, ("async", None, None)),           # ... or fewer, but more than 128 of 256 x 128
    ("bf16", 4224, 1024, 1024, ("persistent narrow", "persistent narrow", None)),   # and of more
]
# the same contractions as 1 x 1 convolutions, whose gradients are always launches of their own
POINTWISE = [
    ("bf16", 609, 392, 1512, (None, "by_k", None)),
    ("bf16", 520, 224, 4192, (None, "by_k split", None)),
    ("bf16", 1217, 1200, 200, (None, None, "by_k")),
]
CONV = [
    # (dtype, h, w, cin, cout, stride, samples, (forward, input gradient, weight gradient))
    ("bf16", 41, 39, 64, 64, 1, 47, ("rows 443", "rows 443", None)),
    ("bf16", 9, 11, 192, 128, 1, 100, ("rows 823", "rows 823", "rows")),
    ("bf16", 20, 20, 64, 64, 1, 100, ("rows 422", "rows 422", None)),
    ("bf16", 14, 14, 128, 72, 1, 90, ("rows 422", None, "by_k split")),
    ("bf16", 16, 16, 136, 136, 1, 20, ("by_k", "by_k", "by_k split")),
    ("f32", 8, 8, 256, 264, 2, 64, (None, None, "by_k")),
    ("f32", 16, 16, 136, 136, 1, 20, ("by_k", "by_k", None)),
    ("bf16", 15, 15, 136, 520, 2, 80, ("async", "by_k", "async split")),
    ("bf16", 33, 6, 192, 80, 1, 55, (None, "async", None)),
]


def _holds(got, want):
    return all(w is None or g == w for g, w in zip(got, want))


@pytest.mark.parametrize("dtype,rows,din,dout,want", DENSE)
def test_route_of_dense_cases(dtype, rows, din, dout, want):
    got = routes.dense_routes(linear(din, dout, False), dtype, rows, 1)
    assert _holds(got, want), got


@pytest.mark.parametrize("dtype,rows,cin,cout,want", POINTWISE)
def test_route_of_pointwise_cases(dtype, rows, cin, cout, want):
    got = routes.pointwise_routes(conv(1, rows, cin, cout, 1, 1, 0, False), dtype, 1, 1)
    assert _holds(got, want), got


@pytest.mark.parametrize("dtype,h,w,cin,cout,stride,samples,want", CONV)
def test_route_of_convolution_cases(dtype, h, w, cin, cout, stride, samples, want):
    got = routes.conv_routes(conv(h, w, cin, cout, 3, stride, 1, False), dtype, samples, 1)
    assert _holds(got, want), got


@pytest.mark.parametrize("case", CONV_ROWS_CASES)
def test_cases_of_the_rows_kernel_reach_it(case):
    h, w, cin, cout, r, micro, N = case
    forward, input_gradient, _ = routes.conv_routes(conv(h, w, cin, cout, r, 1, r // 2, False), "bf16", micro, N)
    assert forward == "rows 1413", forward
    if cout % 64 == 0 and r == 3:
        assert input_gradient.startswith("rows"), input_gradient


@pytest.mark.parametrize("case", CONV_ROWS_WIDE)
def test_cases_of_wider_tiles_reach_them(case):
    h, w, cin, cout, r, micro, N, *want = case
    got = routes.conv_routes(conv(h, w, cin, cout, r, 1, r // 2, False), "bf16", micro, N)
    for g, v in zip(got, want):
        assert (g == "rows %d" % v) if v else not g.startswith("rows"), got


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,rows,din,dout,want", DENSE)
def test_dense(dtype, rows, din, dout, want):
    run_stage_case([linear(din, dout, False)], dtype, rows, 1, seed=rows)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,rows,cin,cout,want", POINTWISE)
def test_pointwise(dtype, rows, cin, cout, want):
    run_stage_case([conv(1, rows, cin, cout, 1, 1, 0, False)], dtype, 1, 1, seed=rows)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,h,w,cin,cout,stride,samples,want", CONV)
def test_convolution(dtype, h, w, cin, cout, stride, samples, want):
    run_stage_case([conv(h, w, cin, cout, 3, stride, 1, False)], dtype, samples, 1, seed=h + cout)
