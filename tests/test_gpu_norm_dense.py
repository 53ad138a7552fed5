"""A layer normalisation and the dense layer behind it in one launch: rows and columns around its 16 x 16 tiles, features around what its four waves
share in one step each and what a row's lanes hold, every epilogue, the normalised rows and statistics that the backward pass reads, and both sides of its rule."""
import numpy as np
import pytest
import torch

from paper_2410_14312_amd import Stage
from tests.test_gpu_stage import _params, run_stage_case
from workloads.configs import layernorm, linear

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d,n,rows,micro", [(8, 1, 1, 1), (24, 17, 5, 3), (40, 15, 16, 2), (64, 192, 32, 8), (56, 33, 31, 3), (64, 16, 17, 1), (72, 48, 9, 2), (120, 100, 7, 5),
                                            (128, 64, 16, 1), (136, 32, 16, 1), (60, 32, 16, 1)])
def test_norm_dense(dtype, d, n, rows, micro):
    run_stage_case([layernorm(d, rows), linear(d, n, False, rows=rows)], dtype, micro, 2, seed=d + n)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d,ffn,rows", [(64, 128, 8), (48, 72, 11)])
def test_epilogues(dtype, d, ffn, rows):
    """Behind the normalisation a GELU (whose argument is kept), a ReLU, and a residual connection of the normalisation's own input."""
    run_stage_case([layernorm(d, rows), linear(d, ffn, False, act="gelu", rows=rows), linear(ffn, d, False, rows=rows), layernorm(d, rows),
                    linear(d, d, True, rows=rows), linear(d, d, False, rows=rows), layernorm(d, rows), linear(d, d, False, rows=rows, skip=1)], dtype, 3, 2, seed=d)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_input_off_by_one_element(dtype):
    """An input that is not on 16 bytes gives what one that is gives, up to the order of the sums."""
    d, n, rows = 64, 32, 9
    specs = [layernorm(d, rows), linear(d, n, False, rows=rows)]
    out = []
    for off in (0, 1):
        gen = np.random.default_rng(3)
        torch.manual_seed(3)
        st = Stage(specs, dtype, 2, 1, 1, 0.1, 0.9, device="cuda:0")
        st.set_params(_params(specs, gen))
        x = torch.randn(2, rows * d, device=st.device).to(st.act_dtype)
        dy = torch.randn(2, rows * n, device=st.device).to(st.act_dtype)
        flat = torch.empty(2 * rows * d + off, dtype=st.act_dtype, device=st.device)
        at = flat[off:].view(2, rows * d)
        at.copy_(x)
        y = torch.empty_like(dy)
        st.forward_micro(0, at, y=y)
        dx = torch.empty_like(x)
        st.backward([0], dy=dy, dx=dx)
        torch.cuda.synchronize()
        out.append((y.float().clone(), dx.float().clone()))
    for a, b in zip(*out):
        assert (a - b).norm() <= (1e-6 if dtype == "f32" else 2 ** -8) * a.norm()
