"""The gradient of a stage input that a residual connection or a join reads: handed over and added by the kernel that writes dx, copied where no other layer
reads the input after it, where dx lies over the upstream gradient, and where the gradient buffers run out."""
import numpy as np
import pytest
import torch

from paper_2410_14312_amd import Stage
from tests.test_gpu_stage import _params, run_stage_case
from workloads.configs import affine, conv, layernorm, linear, resadd, transformer_block

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("s,d,heads,ffn,micro,N", [(8, 32, 1, 64, 1, 2), (32, 64, 2, 128, 4, 4), (64, 128, 2, 512, 4, 2)])
def test_transformer_block(s, d, heads, ffn, micro, N, dtype):
    run_stage_case(transformer_block(s, d, heads, ffn), dtype, micro, N, seed=s + d)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_nested_connections(dtype):
    """Three residual connections open at once, the outermost from the stage input: with it, four buffers do not hold all gradients."""
    d = 32
    specs = [layernorm(d), linear(d, d, False), layernorm(d), linear(d, d, False), layernorm(d), linear(d, d, False, act="gelu"), linear(d, d, False),
             linear(d, d, False, skip=3), linear(d, d, False, skip=6), linear(d, d, False, skip=9)]
    run_stage_case(specs, dtype, 5, 2, seed=5)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_joins(dtype):
    """The input read by a join and a convolution; by a join alone behind one; by two joins."""
    h, c = 6, 16
    body = [conv(h, h, c, c, 3, 1, 1, False), affine(h, h, c, False)]
    run_stage_case(body + [resadd(h, h, c, src_b=3, relu=True)], dtype, 2, 2, seed=6)
    run_stage_case(body + [resadd(h, h, c, src_b=3, relu=False), resadd(h, h, c, src_b=4, relu=True)], dtype, 2, 2, seed=7)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_over_the_upstream_gradient(dtype):
    specs, s, d = transformer_block(16, 64, 1, 128), 16, 64
    out = []
    for same in (False, True):
        gen = np.random.default_rng(9)
        torch.manual_seed(9)
        st = Stage(specs, dtype, 3, 1, 1, 0.1, 0.9, device="cuda:0")
        st.set_params(_params(specs, gen))
        x, dy = (torch.randn(3, s * d, device=st.device).to(st.act_dtype) for _ in range(2))
        dx = dy if same else torch.empty_like(dy)
        st.forward_micro(0, x)
        st.backward([0], dy=dy, dx=dx)
        torch.cuda.synchronize()
        out.append((dx.float().clone(), st.regions[1].view(torch.float32)[st.P:2 * st.P].clone()))
    for a, b in zip(*out):
        assert (a - b).norm() <= (1e-5 if dtype == "f32" else 1e-2) * a.norm()
