"""Max pooling by the winners that the forward pass keeps: windows that overlap, that leave positions out and that reach into the padding, maps that are no
whole number of blocks, channels of a whole piece and not, ties, infinities and NaN, windows of more places than a byte tells apart, one over the whole map among them; and behind
an affine layer, in one pass with its gradient."""
import numpy as np
import pytest
import torch

from paper_2410_14312_amd import Stage
from tests.test_gpu_stage import _params, run_stage_case
from workloads.configs import affine, conv, maxpool

pytestmark = pytest.mark.gpu


def _out(h, k, s, p):
    return (h + 2 * p - k) // s + 1


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("h,w,c,k,stride,pad", [(8, 8, 8, 2, 2, 0), (9, 7, 16, 2, 2, 0), (7, 9, 8, 2, 2, 1), (8, 12, 24, 3, 2, 1), (9, 11, 8, 3, 2, 0), (13, 6, 72, 3, 2, 2),
                                                (10, 10, 8, 2, 3, 0), (9, 9, 8, 3, 1, 1), (6, 6, 12, 3, 2, 1), (7, 5, 3, 2, 2, 0), (5, 5, 8, 5, 2, 2), (26, 24, 8, 11, 2, 3),
                                                (26, 24, 8, 12, 3, 2), (17, 17, 10, 13, 2, 0), (14, 15, 16, 14, 14, 0), (13, 12, 12, 12, 1, 6), (9, 5, 8, 19, 3, 9)])
def test_against_its_definition(dtype, h, w, c, k, stride, pad):
    """Bit for bit in what wins and to rounding in what is summed, with ties, infinities and NaN among the inputs."""
    B, ho, wo = 3, _out(h, k, stride, pad), _out(w, k, stride, pad)
    st = Stage([maxpool(h, w, c, k=k, stride=stride, pad=pad)], dtype, B, 1, 1, 0.1, 0.9, device="cuda:0")
    gen = torch.Generator().manual_seed(h * w + k)
    x = torch.randint(-3, 4, (B, h, w, c), generator=gen).float()
    special = torch.rand(x.shape, generator=gen)
    x[special < 0.02] = float("inf")
    x[(special >= 0.02) & (special < 0.06)] = float("-inf")
    x[(special >= 0.06) & (special < 0.1)] = float("nan")
    x[0, :, :, 0] = float("-inf")
    x[1, :, :, 0] = float("nan")
    dy = torch.randn((B, ho, wo, c), generator=gen).to(st.act_dtype)
    want_y, want_dx = torch.full((B, ho, wo, c), float("-inf")), torch.zeros(B, h, w, c, dtype=torch.float64)
    first = torch.full((B, ho, wo, c), -1, dtype=torch.long)
    for r in range(k):
        for q in range(k):
            for i in range(ho):
                for j in range(wo):
                    a, b = i * stride - pad + r, j * stride - pad + q
                    if 0 <= a < h and 0 <= b < w:
                        better = (x[:, a, b] > want_y[:, i, j]) | (first[:, i, j] < 0)   # (the first place, whatever it holds)
                        now = torch.where(better & ~x[:, a, b].isnan(), x[:, a, b], want_y[:, i, j])
                        want_y[:, i, j] = now
                        first[:, i, j] = torch.where(better, torch.tensor(a * w + b), first[:, i, j])
    flat = want_dx.view(B, h * w, c)
    flat.scatter_add_(1, first.view(B, -1, c), dy.double().view(B, -1, c))
    xd, yd = x.to(st.device).to(st.act_dtype).view(B, -1), torch.empty(B, ho * wo * c, device=st.device, dtype=st.act_dtype)
    dyd, dxd = dy.to(st.device).view(B, -1), torch.empty(B, h * w * c, device=st.device, dtype=st.act_dtype)
    st.forward_micro(0, xd, y=yd)
    st.backward([0], dy=dyd, dx=dxd)
    torch.cuda.synchronize()
    assert torch.equal(yd.float().cpu().view(want_y.shape), want_y)
    got = dxd.double().cpu().view(want_dx.shape)
    # sums of up to ceil(k / stride)^2 terms in fp32, rounded once
    bound = want_dx.abs() * (2 ** -8 if dtype == "bf16" else 2 ** -23) + 2 ** -20 * ((k + stride - 1) // stride) ** 2
    assert ((got - want_dx).abs() <= bound).all()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("h,w,c,k,stride,pad,relu,micro,N", [(8, 8, 8, 3, 2, 1, True, 2, 2), (12, 10, 64, 3, 2, 1, True, 3, 2), (9, 7, 72, 3, 2, 0, True, 1, 3),
                                                             (10, 10, 16, 3, 2, 1, False, 2, 2), (40, 48, 24, 3, 2, 1, True, 4, 2), (8, 8, 8, 2, 2, 0, True, 2, 2),
                                                             (8, 8, 12, 3, 2, 1, True, 2, 2), (8, 8, 5, 3, 2, 1, True, 2, 2), (14, 13, 16, 12, 2, 3, True, 2, 2),
                                                             (14, 13, 16, 12, 2, 3, False, 2, 2)])
def test_behind_an_affine_layer(dtype, h, w, c, k, stride, pad, relu, micro, N):
    ho, wo = _out(h, k, stride, pad), _out(w, k, stride, pad)
    run_stage_case([conv(h, w, 8, c, 3, 1, 1, False), affine(h, w, c, relu), maxpool(h, w, c, k=k, stride=stride, pad=pad), conv(ho, wo, c, 8, 1, 1, 0, False)],
                   dtype, micro, N, seed=h + c, has_pool=True)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_one_pass_and_two(dtype):
    """The pooling and the affine layer in one pass, and (where a caller has the input gradient written over the upstream one) one after the other."""
    h, c = 12, 16
    specs = [conv(h, h, 8, c, 3, 1, 1, False), affine(h, h, c, True), maxpool(h, h, c, k=3, stride=2, pad=1)]
    out = []
    for same in (False, True):
        gen = np.random.default_rng(4)
        torch.manual_seed(4)
        st = Stage(specs, dtype, 3, 1, 1, 0.1, 0.9, device="cuda:0")
        st.set_params(_params(specs, gen))
        x = torch.randn(3, h * h * 8, device=st.device).to(st.act_dtype)
        both = torch.randn(3, h * h * 8, device=st.device).to(st.act_dtype)
        dy = both.view(-1)[:3 * 6 * 6 * c].view(3, -1)
        dx = both if same else torch.empty_like(both)
        st.forward_micro(0, x)
        st.backward([0], dy=dy, dx=dx)
        torch.cuda.synchronize()
        out.append((dx.float().clone(), st.regions[1].view(torch.float32)[st.P:2 * st.P].clone()))
    assert torch.equal(out[0][0], out[1][0])
    assert (out[0][1] - out[1][1]).norm() <= 1e-6 * out[0][1].norm()   # (sums in another order)
