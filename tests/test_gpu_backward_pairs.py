"""Input and weight gradient of a dense layer in one launch, on the small and on the tiled kernel, against the oracle: single rows and
columns, remainders of tiles and of fragments, both halves of a launch longer than the other, masks of ReLU and GELU layers below and a
residual connection's gradient to join; which kernel the sizes take; and weight gradients over many rows against the sums in 64 bits."""
import ctypes as C

import pytest

from paper_2410_14312_amd import load_library
from tests.test_gpu_stage import run_stage_case
from workloads.configs import layernorm, linear

TWO, SMALL, TILED = range(3)


def kind(rows, din, dout, dtype):
    f = getattr(load_library(), "_ZN4tmps13backward_kindEllli")
    return f(C.c_long(rows), C.c_long(din), C.c_long(dout), 2 if dtype == "bf16" else 4)


# rows, input, output features
SIZES = [("f32", 2, 3, 1, SMALL), ("f32", 34, 31, 65, SMALL), ("f32", 236, 100, 10, SMALL), ("f32", 64, 512, 512, SMALL), ("f32", 512, 257, 130, SMALL), ("f32", 64, 1000, 1000, SMALL), ("f32", 300, 17, 530, SMALL),
         ("f32", 256, 1024, 1024, TWO), ("bf16", 2, 1, 3, SMALL), ("bf16", 34, 33, 95, SMALL), ("bf16", 256, 1024, 10, SMALL), ("bf16", 130, 520, 500, SMALL),
         ("bf16", 100, 1000, 1000, SMALL), ("bf16", 236, 1000, 1000, TILED), ("bf16", 512, 776, 712, TILED), ("bf16", 258, 1032, 1096, TILED), ("bf16", 40, 4096, 1024, TILED),
         ("bf16", 1024, 712, 648, TILED), ("bf16", 2048, 1024, 1024, TWO), ("bf16", 1026, 712, 648, TWO), ("bf16", 4096, 1024, 512, TWO), ("bf16", 8116, 24, 1960, TWO),
         ("f32", 916, 1336, 136, SMALL), ("bf16", 2192, 752, 24, SMALL), ("bf16", 4818, 72, 224, SMALL)]


@pytest.mark.parametrize("dtype,rows,din,dout,want", SIZES)
def test_the_rule(dtype, rows, din, dout, want):
    assert kind(rows, din, dout, dtype) == want


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,rows,din,dout,want", [c for c in SIZES if c[-1] != TWO])
def test_both_gradients_in_one_launch(dtype, rows, din, dout, want):
    # (the second layer's input gradient passes the first one's ReLU; the first one's goes to the worker below)
    run_stage_case([linear(24, din, True), linear(din, dout, False)], dtype, rows // 2, 2, seed=rows + din)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,d,ffn,s", [("f32", 36, 72, 6), ("bf16", 40, 88, 5), ("bf16", 264, 712, 64)])
def test_gelu_and_residual_connections(dtype, d, ffn, s):
    run_stage_case([layernorm(d, s), linear(d, ffn, False, act="gelu", rows=s), linear(ffn, d, False, rows=s, skip=2)], dtype, 3, 4, seed=d)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,rows,din,dout", [("bf16", 1024, 712, 648), ("bf16", 4096, 1024, 512), ("bf16", 1921, 1920, 384), ("bf16", 2192, 752, 24), ("bf16", 8116, 24, 1960),
                                                 ("f32", 235, 784, 1000), ("f32", 3432, 108, 112), ("f32", 8059, 24, 4936)])
def test_weight_gradients_over_many_rows(dtype, rows, din, dout):
    """Against the sum of the same products in 64 bits: as far off as a chain of 36 roundings is, 2^-24 sqrt(36 / 6) (2-norm; each is 2^-24 / sqrt(3) of
    the sum so far, whose square grows evenly), or of 4 and one for every 256 rows; a sixth more is allowed.  (One chain over all rows: a rounding for
    every 32 rows in bf16 and for every 8 in fp32.)"""
    import numpy as np
    import torch
    from paper_2410_14312_amd import Stage

    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(rows)
    randn = lambda *shape: torch.randn(*shape, generator=gen, dtype=torch.float32, device="cuda:0")
    st = Stage([linear(din, dout, False)], dtype, rows, 1, 1, 0.1, 0.9, borrow_input=True)
    st.set_params([{"w": (randn(dout, din) / din ** 0.5).cpu().numpy(), "b": np.zeros(dout, np.float32)}])
    x, dy = randn(rows, din).to(st.act_dtype), (randn(rows, dout) / rows).to(st.act_dtype)
    st.forward_micro(0, x)
    st.backward([0], dy=dy, dx=torch.empty_like(x))
    torch.cuda.synchronize()
    got = st.get_grads()[0]["w"]
    want = (dy.double().t().contiguous() @ x.double()).cpu().numpy()
    bound = 7.0 / 6.0 * 2.0 ** -24 * (max(36.0, 4.0 + rows / 256.0) / 6.0) ** 0.5
    assert np.linalg.norm(got - want) < bound * np.linalg.norm(want)
