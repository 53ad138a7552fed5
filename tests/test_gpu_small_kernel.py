"""The small contraction kernel's tiles of 16 x 16, 16 x 32 and 32 x 32 outputs, with eight and with four waves, at their remainders: rows, columns
and k that are no whole tile or step, single ones, a k shorter than a step, and the tile sizes' own limits.  Against the oracle (a stage of one
layer: forward pass, and the weight gradient where it is a launch of its own); which tiles a size takes is asked of the library."""
import ctypes as C

import pytest

from paper_2410_14312_amd import load_library
from tests.test_gpu_stage import run_stage_case
from workloads.configs import linear


class _Plan(C.Structure):
    _fields_ = [("tm", C.c_int), ("tn", C.c_int), ("cost", C.c_double)]


def tiles(M, N, K, dtype):
    f = load_library()._ZN4tmps10small_planEllli
    f.restype = _Plan
    p = f(C.c_long(M), C.c_long(N), C.c_long(K), 2 if dtype == "bf16" else 4)
    return p.tm, p.tn


# rows of a micro-batch, input and output features, tiles of the forward pass
SIZES = [(1, 1, 1, (1, 1)), (16, 16, 16, (1, 1)), (17, 15, 33, (1, 1)), (47, 1000, 1000, (1, 1)), (5, 31, 4081, (1, 1)), (5, 33, 4097, (1, 2)), (256, 7, 256, (1, 1)),
         (241, 70, 273, (1, 2)), (33, 100, 1370, (1, 2)), (250, 63, 260, (1, 2)), (97, 257, 1380, (2, 2)), (256, 1024, 1000, (2, 2)), (500, 12, 510, (2, 2))]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rows,din,dout,want", SIZES)
def test_tiles(dtype, rows, din, dout, want):
    assert tiles(rows, dout, din, dtype) == want


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rows,din,dout,want", SIZES)
def test_small_kernel(dtype, rows, din, dout, want):
    run_stage_case([linear(din, dout, True)], dtype, rows, 1, seed=rows + din + dout)
