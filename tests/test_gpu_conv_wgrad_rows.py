"""Weight gradients of 3 x 3 convolutions on runs of rows: numbers of chunks of 128 positions on both sides of the three that are staged, exact ones and
one position more; one slice and several, of one chunk and of more, the last one shorter; maps of one row and of one column, tiles over many
images, the widest map whose run fits LDS and one wider; several tiles of either channels; fewer positions, which are left to the other kernels.  How many
slices a case makes is asked of the library's rule, with its own estimate of the other kernels, so that a change of the rule cannot quietly empty these tests."""
import numpy as np
import pytest

from tests import routes
from tests.test_gpu_stage import run_stage_case
from workloads.configs import conv

CASES = [
    # (h, w, cin, cout, micro, N, slices; 0: another kernel)
    (2, 2, 512, 512, 31, 1, 0),     # 124 positions
    (4, 4, 512, 512, 8, 1, 0),      # 128
    (3, 43, 512, 512, 1, 1, 0),     # 129
    (2, 2, 64, 64, 300, 1, 10),     # ten slices of one chunk
    (2, 2, 512, 512, 64, 1, 1),     # two chunks
    (257, 1, 512, 512, 1, 1, 1),    # and one position
    (4, 8, 512, 512, 12, 1, 1),     # three
    (7, 11, 512, 512, 5, 1, 1),     # and one position
    (7, 7, 512, 512, 4, 2, 1),      # four, the last one hardly begun
    (8, 8, 64, 192, 30, 1, 8),      # slices
    (1, 61, 128, 128, 33, 1, 8),
    (61, 1, 128, 128, 33, 1, 8),
    (2, 75, 64, 128, 40, 1, 16),
    (2, 76, 64, 128, 40, 1, 0),
    (16, 16, 128, 64, 13, 2, 18),
]


@pytest.mark.gpu
@pytest.mark.parametrize("h,w,cin,cout,micro,N,slices", CASES)
def test_conv_wgrad_rows(h, w, cin, cout, micro, N, slices):
    run_stage_case([conv(h, w, 64, cin, 1, 1, 0, True), conv(h, w, cin, cout, 3, 1, 1, False)], "bf16", micro, N, seed=h + 7 * w + cout)


@pytest.mark.parametrize("h,w,cin,cout,micro,N,slices", CASES + [(16, 16, 128, 72, 13, 2, 0)])
def test_slices_of_the_cases(h, w, cin, cout, micro, N, slices):
    got = routes.conv_wgrad_rows(conv(h, w, cin, cout, 3, 1, 1, False), micro * N)
    assert got.slices == slices
    if slices:
        assert got.per_slice % 128 == 0 and (slices - 1) * got.per_slice < micro * N * h * w <= slices * got.per_slice


# (h, c, samples): those of more than 64 chunks to a slice before they were limited, one just within, one whose other kernel rounds as often
LONG = [(14, 512, 64), (8, 512, 256), (8, 512, 128), (28, 256, 64)]


def roundings(h, c, samples):
    """Of a sum in a wave, two a chunk."""
    return 2 * routes.conv_wgrad_rows(conv(h, h, c, c, 3, 1, 1, False), samples).per_slice // 128


@pytest.mark.parametrize("h,c,samples", LONG)
def test_no_sum_is_rounded_more_often_than_the_other_kernels_would(h, c, samples):
    p = routes.conv_wgrad_plan(conv(h, h, c, c, 3, 1, 1, False), samples)
    chains = 4 if p.kind == 1 else 2 if p.kind == 2 or p.bm * p.bn == 4096 else 1
    n = roundings(h, c, samples)
    assert 0 < n <= max(128, -(-samples * h * h // (16 * p.slices * chains)))


@pytest.mark.gpu
@pytest.mark.parametrize("h,c,samples", LONG)
def test_error_of_long_sums(h, c, samples):
    """Against the sums of the same bf16 products in 64 bits: a sum of random terms rounded n times on its way is 2^-24 sqrt(n / 6) off (2-norm); n is at
    most the 128 or what the other kernels would make, and 4 waves and some slices are added; a twentieth more is allowed."""
    import torch
    from paper_2410_14312_amd import Stage

    spec = conv(h, h, c, c, 3, 1, 1, False)
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(h + c)
    randn = lambda *shape: torch.randn(*shape, generator=gen, device="cuda:0")
    st = Stage([spec], "bf16", samples, 1, 1, 0.1, 0.9, borrow_input=True)
    st.set_params([{"w": (randn(c, 3, 3, c) / (9 * c) ** 0.5).cpu().numpy(), "b": np.zeros(c, np.float32)}])
    x = randn(samples, h, h, c).bfloat16()
    dy = (randn(samples, h, h, c) / samples).bfloat16()
    st.forward_micro(0, x.view(samples, -1))
    st.backward([0], dy=dy.view(samples, -1))
    torch.cuda.synchronize()
    got = torch.from_numpy(st.get_grads()[0]["w"]).to("cuda:0").double()
    padded = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
    d = dy.reshape(-1, c).double().t().contiguous()
    want = torch.stack([d @ padded[:, r:r + h, s:s + h].reshape(-1, c).double() for r in range(3) for s in range(3)], 1).view(c, 3, 3, c)
    p = routes.conv_wgrad_plan(spec, samples)
    n = max(128, -(-samples * h * h // (16 * p.slices * 2))) + 4 + 18
    assert ((got - want).norm() / want.norm()).item() < 1.05 * 2.0 ** -24 * (n / 6) ** 0.5
