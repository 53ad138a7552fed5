"""Stages whose weight and input gradients share launches or wait for the end of the pass, called with the gradient w.r.t. the input
written over the upstream gradient or over the borrowed input: every result equals that of separate buffers (weight gradients to the
order of their fp32 sums, 2^-24 times the root of some thousand terms; the input gradient to one rounding of its type)."""
import numpy as np
import pytest

from workloads.configs import linear

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("over", ["dy", "x"])
@pytest.mark.parametrize("dtype,widths,rows", [("bf16", [768, 2304, 768, 3072, 768], 128), ("f32", [48, 96, 48], 1), ("bf16", [256, 512, 256], 1)])
def test_input_gradient_over_an_operand(dtype, widths, rows, over):
    import torch
    from paper_2410_14312_amd import Stage

    rng = np.random.default_rng(11)
    M = 4 if rows > 1 else 64
    specs = [linear(a, b, False, rows=rows) for a, b in zip(widths, widths[1:])]
    p = [{"w": (rng.standard_normal((b, a)) / np.sqrt(a)).astype(np.float32), "b": rng.standard_normal(b).astype(np.float32)} for a, b in zip(widths, widths[1:])]
    x = rng.standard_normal((M, rows * widths[0])).astype(np.float32)
    dy = (rng.standard_normal((M, rows * widths[-1])) / M).astype(np.float32)
    got = []
    for alias in (False, True):
        st = Stage(specs, dtype, M, 1, 1, 0.1, 0.9, borrow_input=True)
        st.set_params(p)
        xd, dyd = (torch.from_numpy(a).to(st.act_dtype).to(st.device) for a in (x, dy))
        dx = (dyd if over == "dy" else xd) if alias else torch.empty_like(xd)
        st.forward_micro(0, xd)
        st.backward([0], dy=dyd, dx=dx)
        torch.cuda.synchronize()
        got.append((st.get_grads(), dx.float().cpu().numpy()))
    for a, b in zip(got[0][0], got[1][0]):
        for k in a:
            assert np.linalg.norm(a[k] - b[k]) < 1e-5 * np.linalg.norm(a[k])
    assert np.linalg.norm(got[0][1] - got[1][1]) < (1e-5 if dtype == "f32" else 2.0 ** -9) * np.linalg.norm(got[0][1])
