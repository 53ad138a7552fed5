"""What a stage's forward pass hands to the next worker leaves the last contraction in two places, the caller's and the stash: the same bytes in both, on every
kind of kernel that ends a stage (small, tiled, split along k, persistent; with a residual connection, an affine layer, a join; fp32 logits), with
the caller's at a 16-byte address and at one that is not, and over the pass's own input, where it is copied afterwards."""
import numpy as np
import pytest
import torch

from paper_2410_14312_amd import Stage
from tests.test_gpu_stage import _params as make_params
from workloads.configs import affine, bottleneck, conv, layernorm, linear, maxpool, softmax_ce

pytestmark = pytest.mark.gpu

STAGES = {
    "small": [linear(64, 128, True)],
    "ragged": [linear(61, 83, False)],
    "split": [linear(3072, 96, False)],
    "persistent": [linear(256, 256, False, rows=512)],
    "residual": [layernorm(128, 64), linear(128, 512, False, rows=64, act="gelu"), linear(512, 128, False, rows=64, skip=2)],
    "affine": [conv(8, 8, 16, 24, 3, 1, 1, False), affine(8, 8, 24, True)],
    "join": [conv(6, 6, 8, 32, 1, 1, 0, True)] + bottleneck(6, 32, 8, 1, False)[0],
    "pool": [conv(8, 8, 8, 16, 3, 1, 1, True), maxpool(8, 8, 16)],
    "logits": [linear(64, 1003, False), softmax_ce(1003)],
    "wide logits": [linear(64, 5003, False, rows=40), softmax_ce(5003, rows=40)],
}


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("name", sorted(STAGES))
def test_both_places(name, dtype):
    specs, micro = STAGES[name], 96
    gen = np.random.default_rng(7)
    st = Stage(specs, dtype, micro, 2, 2, 0.1, 0.9, borrow_input=True, device="cuda:0")
    st.set_params(make_params(specs, gen))
    x = torch.randn(micro, st.in_elems, device=st.device).to(st.act_dtype)
    labels = torch.zeros(micro, specs[-1].get("rows", 1), dtype=torch.int32, device=st.device) if st.is_last else None
    ydt = torch.float32 if st.is_last else st.act_dtype
    n = micro * st.out_elems
    room = torch.full((n + 16,), -7.0, device=st.device, dtype=ydt)
    for slot, first in ((0, 0), (1, 1)):   # on a 16-byte address and one element further
        room.fill_(-7.0)
        st.forward_micro(slot, x, y=room[first:first + n], labels=labels)
        torch.cuda.synchronize()
        nbytes = n * room.element_size()
        kept = torch.empty(nbytes, dtype=torch.uint8, device=st.device)
        base = st.regions[2].data_ptr()
        off = st.output_ptr(slot) - base
        kept.copy_(st.regions[2][off:off + nbytes])
        assert torch.equal(kept.view(ydt), room[first:first + n])
        assert (room[:first] == -7.0).all() and (room[first + n:] == -7.0).all()


def test_over_the_input():
    specs, micro = [linear(64, 64, False)], 48
    gen = np.random.default_rng(8)
    st = Stage(specs, "f32", micro, 1, 1, 0.1, 0.9, borrow_input=True, device="cuda:0")
    st.set_params(make_params(specs, gen))
    x = torch.randn(micro, 64, device=st.device, dtype=torch.float32)
    ref, both = torch.empty_like(x), x.clone()
    st.forward_micro(0, x, y=ref)
    torch.cuda.synchronize()
    st = Stage(specs, "f32", micro, 1, 1, 0.1, 0.9, borrow_input=True, device="cuda:0")
    gen = np.random.default_rng(8)
    st.set_params(make_params(specs, gen))
    st.forward_micro(0, both, y=both)
    torch.cuda.synchronize()
    assert torch.equal(ref, both)
