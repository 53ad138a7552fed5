"""Weight gradients of several dense layers in one persistent launch: stages whose layers the rule groups, with tiles that end in whole rounds of
the device, tiles cut along k, and ragged last tiles, against the oracle; the rule itself on the CPU."""
import ctypes as C

import numpy as np
import pytest

from paper_2410_14312_amd import load_library
from tests.test_gpu_stage import run_stage_case
from workloads.configs import layernorm, linear, softmax_ce, transformer_block

PART = 256 * 128 + 256   # floats of a partial tile


def group_elems(widths, rows):
    f = getattr(load_library(), "_ZN4tmps23dense_wgrad_group_elemsElPA2_Kii")
    f.restype = C.c_int64
    dims = [v for a, b in zip(widths, widths[1:]) for v in (a, b)]
    return f(C.c_int64(rows), (C.c_int * len(dims))(*dims), len(dims) // 2)


# widths, rows, partial tiles: none; 128 tiles in two slices; a ragged last tile in both directions; more than two rounds; a whole round and 64 tiles in
# two slices; the same with ragged ones among them; 25 k-tiles, which chains of 4 do not divide, in slices of 13 and 12
CASES = [([768, 2304, 768, 3072, 768], 512, 0), ([1024] * 5, 4096, 256), ([1032, 2048, 776, 1288], 2048, None), ([1024] * 21, 1024, None),
         ([1024] * 11, 1024, 128), ([1032, 1040, 776] * 3 + [1032], 1024, 184), ([1024] * 5, 1600, 256)]


@pytest.mark.parametrize("widths,rows,parts", CASES)
def test_the_rule_groups_them(widths, rows, parts):
    n = group_elems(widths, rows)
    assert n >= 0 and n % PART == 0 and (parts is None or n == parts * PART)


def test_the_rule_leaves_few_or_short_ones_alone():
    assert group_elems([512, 512], 1024) == -1 and group_elems([256, 512, 256], 512) == -1


@pytest.mark.gpu
@pytest.mark.parametrize("widths,rows,parts", CASES)
def test_grouped_weight_gradients(widths, rows, parts):
    run_stage_case([linear(a, b, False, rows=rows // 4) for a, b in zip(widths, widths[1:])], "bf16", 2, 2, seed=rows, deep=len(widths) > 10)


# rows, k-tiles of 64 that are summed in one go
CHAINS = [(512, 2), (960, 2), (1024, 4), (1600, 4), (4032, 4), (4096, 8), (8192, 8)]


@pytest.mark.gpu
@pytest.mark.parametrize("rows,chain", CHAINS)
def test_long_sums_are_as_exact_as_short_ones(rows, chain):
    """The last layer's gradient of a group against the sum of the same bf16 products in 64 bits.  A sum of random terms that takes n roundings on its
    way is 2^-24 sqrt(n / 6) from it (each rounding 2^-24 / sqrt(3) of the sum so far, whose square grows evenly): a chain of `chain` k-tiles takes four
    roundings a k-tile, the sum of the chains one each; a quarter more is allowed."""
    import torch
    from paper_2410_14312_amd import Stage

    widths = [768, 2304, 768, 3072, 768]
    assert group_elems(widths, rows) >= 0
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(rows)
    randn = lambda *shape: torch.randn(*shape, generator=gen, device="cuda:0")
    specs = [linear(a, b, False) for a, b in zip(widths, widths[1:])]
    p = [{"w": (randn(b, a) / a ** 0.5).cpu().numpy(), "b": np.zeros(b, np.float32)} for a, b in zip(widths, widths[1:])]
    x = randn(rows, widths[0]).bfloat16()
    dy = (randn(rows, widths[-1]) / rows).bfloat16()
    below = Stage(specs[:-1], "bf16", rows, 1, 1, 0.1, 0.9, borrow_input=True)   # (the last layer's input)
    below.set_params(p[:-1])
    mid = torch.empty(rows, widths[-2], dtype=torch.bfloat16, device="cuda:0")
    below.forward_micro(0, x, y=mid)
    st = Stage(specs, "bf16", rows, 1, 1, 0.1, 0.9, borrow_input=True)
    st.set_params(p)
    st.forward_micro(0, x)
    st.backward([0], dy=dy)
    torch.cuda.synchronize()
    got = st.get_grads()[-1]
    want = (dy.double().t().contiguous() @ mid.double()).cpu().numpy()
    bound = 1.25 * 2.0 ** -24 * ((4 * chain + rows / 64 / chain) / 6) ** 0.5
    assert np.linalg.norm(got["w"] - want) < bound * np.linalg.norm(want)
    want = dy.double().sum(0).cpu().numpy()
    assert np.linalg.norm(got["b"] - want) < bound * np.linalg.norm(want)


@pytest.mark.gpu
def test_grouped_behind_residual_connections_and_the_loss():
    s, d, vocab = 256, 768, 1024
    specs = transformer_block(s, d, 12, 3072) + [layernorm(d, s), linear(d, vocab, False, rows=s), softmax_ce(vocab, rows=s)]
    assert group_elems([d, vocab], 512) == -1
    run_stage_case(specs, "bf16", 1, 2, seed=3)


@pytest.mark.gpu
def test_an_operand_at_an_odd_address_is_left_out_of_the_group():
    """Borrowed input 2 bytes off a 16-byte boundary: that layer's gradient is a launch of its own, the others' still one."""
    import torch
    from paper_2410_14312_amd import Stage

    rng = np.random.default_rng(5)
    widths, rows, M = [768, 2304, 768, 3072, 768], 128, 4
    specs = [linear(a, b, False, rows=rows) for a, b in zip(widths, widths[1:])]
    p = [{"w": (rng.standard_normal((b, a)) / np.sqrt(a)).astype(np.float32), "b": rng.standard_normal(b).astype(np.float32)} for a, b in zip(widths, widths[1:])]
    x = rng.standard_normal((M, rows * widths[0])).astype(np.float32)
    dy = (rng.standard_normal((M, rows * widths[-1])) / M).astype(np.float32)
    got = []
    for odd in (0, 1):
        st = Stage(specs, "bf16", M, 1, 1, 0.1, 0.9, borrow_input=True)
        st.set_params(p)
        flat = torch.zeros(x.size + 8, dtype=torch.bfloat16, device=st.device)
        xd = flat[odd:odd + x.size].view(M, -1)
        xd.copy_(torch.from_numpy(x))
        st.forward_micro(0, xd)
        st.backward([0], dy=torch.from_numpy(dy).to(torch.bfloat16).to(st.device))
        torch.cuda.synchronize()
        got.append(st.get_grads())
    for a, b in zip(*got):
        for k in a:   # (the forward pass takes another kernel for such an input: sums in another order, then bf16 rounding)
            assert np.linalg.norm(a[k] - b[k]) < 1e-2 * np.linalg.norm(a[k])
