"""Weight gradients of several dense layers in one persistent launch: stages whose layers the rule groups, with tiles that end in whole rounds of
the device, tiles cut along k, and ragged last tiles, against the oracle; the rule itself on the CPU."""
import ctypes as C

import numpy as np
import pytest

from paper_2410_14312_amd import load_library
from tests.test_gpu_stage import run_stage_case
from workloads.configs import layernorm, linear, softmax_ce, transformer_block

PART = 256 * 256 + 256   # floats of a partial tile


def group_elems(widths, rows):
    f = getattr(load_library(), "_ZN4tmps23dense_wgrad_group_elemsElPA2_Kii")
    f.restype = C.c_int64
    dims = [v for a, b in zip(widths, widths[1:]) for v in (a, b)]
    return f(C.c_int64(rows), (C.c_int * len(dims))(*dims), len(dims) // 2)


# widths, rows, partial tiles: none; 40 of 42 tiles' slices; a ragged last tile in both directions; a whole round and 64 tiles in two slices
CASES = [([768, 2304, 768, 3072, 768], 512, 0), ([1024] * 5, 4096, 256), ([1032, 2048, 776, 1288], 2048, None), ([1024] * 21, 1024, 128)]


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
