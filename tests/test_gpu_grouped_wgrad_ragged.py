"""Grouped weight gradients over rows that are no multiple of 64: one row and 63 in the last k-tile, whole rounds and tiles in slices (the last slice
alone has a short k-tile), ragged tiles; the rule on the CPU.  What lies behind the last row is filled with NaN."""
import numpy as np
import pytest

from tests.test_gpu_grouped_wgrad import group_elems
from workloads.configs import linear

# widths, rows, partial tiles
CASES = [([768, 2304, 768, 3072, 768], 513, 0), ([768, 2304, 768, 3072, 768], 575, 0), ([1024] * 5, 4100, 256), ([1032, 2048, 776, 1288], 2047, None),
         ([1024] * 11, 1001, 128)]


@pytest.mark.parametrize("widths,rows,parts", CASES)
def test_the_rule_groups_them(widths, rows, parts):
    n = group_elems(widths, rows)
    assert n >= 0 and (parts is None or n == parts * (256 * 128 + 256))


@pytest.mark.gpu
@pytest.mark.parametrize("widths,rows,parts", CASES)
def test_against_64_bits(widths, rows, parts):
    """The last and the first layer's gradients (of a stage of dense layers without activation) against sums of the same bf16 products in 64 bits, within
    what the chains of test_gpu_grouped_wgrad.py allow; both operands of the last layer end where NaN begins."""
    import torch
    from paper_2410_14312_amd import Stage

    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(rows)
    randn = lambda *shape: torch.randn(*shape, generator=gen, device="cuda:0", dtype=torch.float32)
    specs = [linear(a, b, False) for a, b in zip(widths, widths[1:])]
    p = [{"w": (randn(b, a) / a ** 0.5).cpu().numpy(), "b": np.zeros(b, np.float32)} for a, b in zip(widths, widths[1:])]

    def padded(v):
        flat = torch.full((v.numel() + 64 * v.shape[1],), float("nan"), dtype=torch.bfloat16, device="cuda:0")
        flat[:v.numel()] = v.flatten().bfloat16()
        return flat[:v.numel()].view(v.shape)

    x, dy = padded(randn(rows, widths[0])), padded(randn(rows, widths[-1]) / rows)
    below = Stage(specs[:-1], "bf16", rows, 1, 1, 0.1, 0.9, borrow_input=True)   # (the last layer's input)
    below.set_params(p[:-1])
    mid = torch.empty(rows, widths[-2], dtype=torch.bfloat16, device="cuda:0")
    below.forward_micro(0, x, y=mid)
    above = Stage(specs[1:], "bf16", rows, 1, 1, 0.1, 0.9, borrow_input=True)   # (the gradient of the first layer's result)
    above.set_params(p[1:])
    first = torch.empty(rows, widths[1], dtype=torch.bfloat16, device="cuda:0")
    first_in = torch.empty(rows, widths[1], dtype=torch.bfloat16, device="cuda:0")
    one = Stage(specs[:1], "bf16", rows, 1, 1, 0.1, 0.9, borrow_input=True)
    one.set_params(p[:1])
    one.forward_micro(0, x, y=first_in)
    above.forward_micro(0, first_in)
    above.backward([0], dy=dy, dx=first)
    st = Stage(specs, "bf16", rows, 1, 1, 0.1, 0.9, borrow_input=True)
    st.set_params(p)
    st.forward_micro(0, x)
    st.backward([0], dy=dy)
    torch.cuda.synchronize()
    kt = (rows + 63) // 64
    chain = 2 if kt < 16 else 4 if kt < 64 else 8
    bound = 1.25 * 2.0 ** -24 * ((4 * chain + kt / chain) / 6) ** 0.5
    for got, g, v in ((st.get_grads()[-1], dy, mid), (st.get_grads()[0], first, x)):
        want = (g.double().t().contiguous() @ v.double()).cpu().numpy()
        assert np.linalg.norm(got["w"] - want) < bound * np.linalg.norm(want)
        want = g.double().sum(0).cpu().numpy()
        assert np.linalg.norm(got["b"] - want) < bound * np.linalg.norm(want)
