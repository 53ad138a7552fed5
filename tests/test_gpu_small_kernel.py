"""The small contraction kernel's tiles of 16 x 16, 16 x 32 and 32 x 32 outputs, with eight and with four waves, at their remainders: rows, columns
and k that are no whole tile or step, single ones, a k shorter than a step, and the tile sizes' own limits.  Against the oracle (a stage of one
layer: forward pass, and the weight gradient where it is a launch of its own); which tiles a size takes is asked of the library.
And the forward pass in fp32 against the sums in 64 bits."""
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


@pytest.mark.gpu
@pytest.mark.parametrize("rows,din,dout", [(47, 1000, 1000), (235, 1000, 1000), (256, 1024, 1000), (33, 1370, 100), (16, 1600, 16)])
def test_sums_of_long_contractions(rows, din, dout):
    """Chains of at most 16 roundings (six steps of one multiply, two roundings each, for each of four accumulators, and their sum), one for every six
    steps of a wave and one for every wave: as far from the sum in 64 bits as a chain of 28, 2^-24 sqrt(28 / 6) (2-norm; each rounding is 2^-24 / sqrt(3)
    of the sum so far, whose square grows evenly).  One chain to a wave: twice as many and more, from 1000 features on."""
    import numpy as np
    import torch
    from paper_2410_14312_amd import Stage

    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(din)
    f32 = dict(dtype=torch.float32, device="cuda:0")
    w = torch.randn(dout, din, generator=gen, **f32) / din ** 0.5
    x = torch.randn(rows, din, generator=gen, **f32)
    st = Stage([linear(din, dout, False)], "f32", rows, 1, 1, 0.1, 0.9, borrow_input=True)
    st.set_params([{"w": w.cpu().numpy(), "b": np.zeros(dout, np.float32)}])
    y = torch.empty(rows, dout, **f32)
    st.forward_micro(0, x, y=y)
    want = x.double() @ w.double().t().contiguous()
    assert (y.double() - want).norm() < 2.0 ** -24 * (28 / 6) ** 0.5 * want.norm()
