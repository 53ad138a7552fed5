"""A 1 x 1 convolution and the affine layer behind it, forward to twice and four times as many channels and their gradients in one pass: every pair of widths, positions that end inside a step of 64, a piece of 16 and a
workgroup's run, with and without ReLU below, a gradient to join; against sums of the same bf16 values in 64 bits."""
import ctypes as C

import numpy as np
import pytest

from paper_2410_14312_amd import load_library
from workloads.configs import affine, conv

WIDTHS = [(64, 64), (64, 128), (128, 64), (128, 128), (64, 256), (256, 64)]   # out of the convolution, into it
# samples, height, width of the map: 1024 positions, 16 to a workgroup, and one more; 16384, 80 to a workgroup; a last one with fewer, off 16
MAPS = [(1, 32, 32), (1, 25, 41), (4, 64, 64), (7, 49, 51), (16, 35, 36)]


def takes(P, O, I, dtype=1):
    f = getattr(load_library(), "_ZN4tmps22affine_pointwise_takesEilii")
    f.restype, f.argtypes = C.c_bool, [C.c_int, C.c_long, C.c_int, C.c_int]
    return f(dtype, P, O, I)


def test_the_rule():
    assert all(takes(1024, o, i) for o, i in WIDTHS)
    assert not takes(1023, 64, 64) and not takes(20000, 128, 256) and not takes(20000, 96, 64) and not takes(20000, 512, 64) and not takes(20000, 64, 64, 0)


@pytest.mark.gpu
@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("B,h,w", MAPS)
@pytest.mark.parametrize("cout,cin", WIDTHS)
def test_against_64_bits(cout, cin, B, h, w, relu):
    import torch
    from paper_2410_14312_amd import Stage

    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(cout + cin + h)
    randn = lambda *shape: torch.randn(*shape, generator=gen, device="cuda:0", dtype=torch.float32)
    P = B * h * w
    # (with ReLU the convolution reads another's result, through which its input gradient passes: a 1 x 1 layer of 8 channels)
    specs = ([conv(h, w, 8, cin, 1, 1, 0, True)] if relu else []) + [conv(h, w, cin, cout, 1, 1, 0, False), affine(h, w, cout, False)]
    p = ([{"w": randn(cin, 1, 1, 8) / 8 ** 0.5, "b": 0.1 * randn(cin)}] if relu else []) + [
        {"w": randn(cout, 1, 1, cin) / cin ** 0.5, "b": 0.1 * randn(cout)}, {"w": 1 + 0.2 * randn(cout), "b": 0.1 * randn(cout)}]
    st = Stage(specs, "bf16", B, 1, 1, 0.1, 0.9, borrow_input=True)
    st.set_params([{k: v.cpu().numpy() for k, v in q.items()} for q in p])
    x = randn(B, h * w * (8 if relu else cin)).bfloat16()
    dy = (randn(B, h * w * cout) / P).bfloat16()
    dx = torch.full_like(x, float("nan"))
    st.forward_micro(0, x)
    st.backward([0], dy=dy, dx=dx)
    torch.cuda.synchronize()
    got = st.get_grads()
    d64 = lambda t: t.double()
    xin = x.view(P, -1)
    if relu:   # the stored activation: fp32 sums of eight products, rounded
        xin = torch.relu(d64(xin) @ d64(p[0]["w"].view(cin, 8).bfloat16()).t() + d64(p[0]["b"])).bfloat16()
    wb = p[-2]["w"].view(cout, cin).bfloat16()
    z = (d64(xin) @ d64(wb).t() + d64(p[-2]["b"])).bfloat16()
    g = (dy.view(P, cout).float() * p[-1]["w"]).bfloat16()
    rel = lambda a, b: float(torch.linalg.norm(d64(torch.as_tensor(a).to(b.device)) - b) / torch.linalg.norm(b))
    # z and x may differ from the stored ones by a rounding here and there: 2^-9 of a value in one of some thousand
    assert rel(got[-1]["w"], (d64(dy.view(P, cout)) * d64(z)).sum(0)) < 1e-4
    assert rel(got[-1]["b"], d64(dy.view(P, cout)).sum(0)) < 5e-7
    assert rel(got[-2]["b"], d64(g).sum(0)) < 5e-7
    want = d64(g).t().contiguous() @ d64(xin)
    assert rel(got[-2]["w"].reshape(cout, cin), want) < (1e-4 if relu else 2.5e-7)
    if not relu:
        want = d64(g) @ d64(wb)
        assert rel(dx.view(P, cin), want) < 2.0 ** -8.5
        assert float((d64(dx.view(P, cin)) - want).abs().max() / want.abs().max()) < 2.0 ** -8
    else:
        # stored in bf16: one value in some thousand is rounded to the other side, by 2^-8 of it, 2^-8 / sqrt(1000) of the whole in the 2-norm
        below = d64(((d64(g) @ d64(wb)) * (xin > 0)).bfloat16())
        assert rel(got[0]["w"].reshape(cin, 8), below.t().contiguous() @ d64(x.view(P, 8))) < 2.5e-4
        assert rel(got[0]["b"], below.sum(0)) < 2.5e-4


@pytest.mark.gpu
@pytest.mark.parametrize("h,micro", [(32, 8), (37, 3), (64, 1), (31, 4)])
def test_bottleneck_blocks_against_the_oracle(h, micro):
    """Both 1 x 1 convolutions of a block with a projection and of two without, whose shortcut's gradient the first one joins; forward the join and the next
    block's first convolution leave one launch (from 4096 positions of a micro-batch on), with positions off 16 and 64, and the projection and the last join theirs."""
    from tests.test_gpu_stage import run_stage_case
    from workloads.configs import bottleneck

    specs, c = [], 64
    for k in range(3):
        block, h, c = bottleneck(h, c, 64, 1, k == 0)
        specs += block
    run_stage_case(specs, "bf16", micro, 2, seed=11, deep=True)


@pytest.mark.gpu
@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("B,h,w", [(1, 64, 64), (3, 37, 37), (1, 71, 103), (5, 60, 60)])
def test_forward_is_as_its_layers_round(B, h, w, relu):
    """64 channels to 256 with the affine layer: sums in 64 bits, rounded where the layers store; beside them only neighbours of a rounding may differ."""
    import torch
    from paper_2410_14312_amd import Stage

    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(h + w)
    randn = lambda *shape: torch.randn(*shape, generator=gen, device="cuda:0", dtype=torch.float32)
    P = B * h * w
    wt, bias, gain, shift = randn(256, 1, 1, 64) / 8, 0.1 * randn(256), 1 + 0.2 * randn(256), 0.1 * randn(256)
    st = Stage([conv(h, w, 64, 256, 1, 1, 0, False), affine(h, w, 256, relu)], "bf16", B, 1, 1, 0.1, 0.9, borrow_input=True)
    st.set_params([{"w": wt.cpu().numpy(), "b": bias.cpu().numpy()}, {"w": gain.cpu().numpy(), "b": shift.cpu().numpy()}])
    x = randn(B, h * w * 64).bfloat16()
    y = torch.full((B, h * w * 256), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    st.forward_micro(0, x, y=y)
    torch.cuda.synchronize()
    z = (x.view(P, 64).double() @ wt.view(256, 64).bfloat16().double().t() + bias.double()).bfloat16()
    want = gain.double() * z.double() + shift.double()
    want = (torch.relu(want) if relu else want).bfloat16()
    got = y.view(P, 256)
    assert float((got != want).double().mean()) < 1e-3
    # (a z on the other side of its rounding, 2^-8 of it, times a gain below 2, and y's own rounding)
    assert float(((got.double() - want.double()).abs() - 2.0 ** -7 * (z.double().abs() * 2 + want.double().abs())).max()) <= 0


FORWARD = [(32, 64), (32, 128), (64, 128), (64, 256)]   # into the convolution, out of it


def forward_takes(P, I, O, following):
    f = getattr(load_library(), "_ZN4tmps23pointwise_forward_takesEliib")
    f.restype, f.argtypes = C.c_bool, [C.c_long, C.c_int, C.c_int, C.c_bool]
    return f(P, I, O, following)


def test_the_rule_of_the_forward_pass():
    for i, o in FORWARD:
        assert forward_takes(4096, i, o, False) and forward_takes(256, i, o, True) and not forward_takes(4095, i, o, False) and not forward_takes(255, i, o, True)
        assert not forward_takes(20000, o, i, False) and not forward_takes(20000, i, i, True)
    assert not forward_takes(20000, 128, 256, False) and not forward_takes(20000, 128, 512, True) and not forward_takes(20000, 16, 64, False)


@pytest.mark.gpu
@pytest.mark.parametrize("B,h,w", [(1, 64, 64), (5, 37, 37), (2, 120, 73)])
@pytest.mark.parametrize("cin,cout", FORWARD)
def test_forward_of_every_pair_of_widths(cin, cout, B, h, w):
    """Sums in 64 bits, rounded where the layers store, with a second place for the result: beside them only neighbours of a rounding may differ."""
    import torch
    from paper_2410_14312_amd import Stage

    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(h + w + cin + cout)
    randn = lambda *shape: torch.randn(*shape, generator=gen, device="cuda:0", dtype=torch.float32)
    P = B * h * w
    wt, bias, gain, shift = randn(cout, 1, 1, cin) / cin ** 0.5, 0.1 * randn(cout), 1 + 0.2 * randn(cout), 0.1 * randn(cout)
    st = Stage([conv(h, w, cin, cout, 1, 1, 0, False), affine(h, w, cout, True)], "bf16", B, 1, 1, 0.1, 0.9, borrow_input=True)
    st.set_params([{"w": wt.cpu().numpy(), "b": bias.cpu().numpy()}, {"w": gain.cpu().numpy(), "b": shift.cpu().numpy()}])
    x = randn(B, h * w * cin).bfloat16()
    y = torch.full((B, h * w * cout), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    st.forward_micro(0, x, y=y)
    torch.cuda.synchronize()
    z = (x.view(P, cin).double() @ wt.view(cout, cin).bfloat16().double().t() + bias.double()).bfloat16()
    want = torch.relu(gain.double() * z.double() + shift.double()).bfloat16()
    got = y.view(P, cout)
    assert float((got != want).double().mean()) < 1e-3
    # (a z on the other side of its rounding, 2^-8 of it, times a gain below 2, and y's own rounding)
    assert float(((got.double() - want.double()).abs() - 2.0 ** -7 * (z.double().abs() * 2 + want.double().abs())).max()) <= 0


@pytest.mark.gpu
@pytest.mark.parametrize("h,w,micro", [(16, 16, 1), (17, 19, 1), (8, 9, 4), (64, 65, 1), (15, 17, 1)])
@pytest.mark.parametrize("cin,cout", FORWARD)
def test_join_and_the_next_convolution_of_every_pair_of_widths(cin, cout, h, w, micro):
    """From 256 positions of a micro-batch on in one launch (the last case: 255), with positions off 16, 32 and 64."""
    from tests.test_gpu_stage import run_stage_case
    from workloads.configs import resadd

    block = [conv(h, w, cout, cin, 1, 1, 0, False), affine(h, w, cin, True), conv(h, w, cin, cout, 1, 1, 0, False), affine(h, w, cout, False, init_gain=0.2),
             resadd(h, w, cout, src_b=5, relu=True)]
    run_stage_case([conv(h, w, 8, cout, 1, 1, 0, True)] + block + block[:2] + [conv(h, w, cin, 8, 1, 1, 0, False)], "bf16", micro, 2, seed=h + cin + cout, deep=True)
