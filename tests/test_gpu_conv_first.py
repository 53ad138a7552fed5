"""Convolutions over eight channels (a padded RGB image, or eight channels of a network's own): tiles of 8 x 16 positions that are full, ragged in
either direction and larger than the map; even and odd maps, padding that lies outside, inside and absent; columns of the result that fill 64, a part
of them and more than them; one tile to a workgroup of the weight gradient, several, and a last one with fewer."""
import pytest

from tests import routes
from tests.test_gpu_stage import run_stage_case
from workloads.configs import affine, conv

CASES = [
    # (h, w, cin, cout, r, stride, pad, micro, N, kinds of the forward pass and of the weight gradient)
    (8, 16, 3, 64, 3, 1, 1, 1, 1, (1, 1)),
    (1, 1, 3, 8, 3, 1, 1, 3, 1, (1, 1)),
    (9, 17, 3, 64, 3, 1, 1, 2, 2, (1, 1)),
    (7, 15, 8, 24, 3, 1, 0, 3, 1, (1, 1)),
    (32, 32, 3, 72, 3, 1, 2, 2, 2, (1, 1)),
    (33, 47, 3, 40, 3, 1, 1, 24, 1, (1, 1)),     # more tiles than workgroups
    (8, 40, 8, 136, 3, 1, 1, 70, 1, (1, 1)),     # three column blocks
    (16, 32, 3, 64, 7, 2, 3, 15, 1, (0, 0)),
    (16, 32, 3, 64, 7, 2, 3, 16, 1, (2, 0)),
    (7, 7, 3, 16, 7, 2, 0, 255, 1, (2, 0)),
    (7, 7, 3, 16, 7, 2, 0, 256, 1, (2, 2)),      # one position, a tile to a workgroup
    (5, 3, 3, 64, 7, 2, 3, 130, 2, (2, 2)),
    (37, 65, 3, 64, 7, 2, 3, 15, 2, (2, 2)),
    (64, 99, 8, 48, 7, 2, 3, 24, 1, (2, 2)),
    (50, 50, 3, 80, 7, 2, 4, 30, 2, (2, 2)),
]


def padded(h, w, cin, cout, r, stride, pad):
    return conv(h, w, 8, cout, r, stride, pad, True)


@pytest.mark.gpu
@pytest.mark.parametrize("h,w,cin,cout,r,stride,pad,micro,N,kinds", CASES)
def test_conv_first(h, w, cin, cout, r, stride, pad, micro, N, kinds):
    run_stage_case([conv(h, w, cin, cout, r, stride, pad, True)], "bf16", micro, N, seed=h + 7 * w + cout)


@pytest.mark.gpu
@pytest.mark.parametrize("h,w,cout,r,stride,pad", [(19, 33, 64, 7, 2, 3), (11, 18, 40, 3, 1, 1)])
def test_with_an_affine_layer(h, w, cout, r, stride, pad):
    ho, wo = ((n + 2 * pad - r) // stride + 1 for n in (h, w))
    run_stage_case([conv(h, w, 3, cout, r, stride, pad, False), affine(ho, wo, cout, True)], "bf16", 70, 1, seed=h + cout)


@pytest.mark.gpu
@pytest.mark.parametrize("h,w,cout,r,stride,pad", [(21, 30, 64, 7, 2, 3), (9, 20, 24, 3, 1, 1)])
def test_inside_a_network(h, w, cout, r, stride, pad):
    """(its input gradient is the other kernels')"""
    run_stage_case([conv(h, w, 16, 8, 1, 1, 0, True), conv(h, w, 8, cout, r, stride, pad, False)], "bf16", 70, 1, seed=w + cout)


@pytest.mark.gpu
@pytest.mark.parametrize("r,stride,pad", [(3, 1, 1), (7, 2, 3)])
def test_infinities_stay_where_they_are_read(r, stride, pad):
    """A pixel that only positions past the edge of a tile would pair with a tap that the map's own positions do not: the last column."""
    import numpy as np
    import torch
    from paper_2410_14312_amd import Stage

    h, w, cout, n = 12, 20, 16, 130
    spec = conv(h, w, 3, cout, r, stride, pad, False)
    gen = np.random.default_rng(5)
    x = gen.standard_normal((n, h, w, 3)).astype(np.float32)
    x[0, 3, w - 1, 1] = np.inf
    wt = gen.standard_normal((cout, r, r, 3)).astype(np.float32)
    st = Stage([spec], "bf16", n, 1, 1, 0.1, 0.9, device="cuda:0")
    st.set_params([{"w": wt, "b": np.zeros(cout, np.float32)}])
    y = torch.empty(n, st.out_elems, dtype=st.act_dtype, device=st.device)
    st.forward_micro(0, st.prepare_input(x), y=y)
    st.backward([0], dy=torch.ones_like(y))
    torch.cuda.synchronize()
    ref = torch.nn.functional.conv2d(torch.from_numpy(x).bfloat16().float().permute(0, 3, 1, 2), torch.from_numpy(wt).bfloat16().float().permute(0, 3, 1, 2),
                                     stride=stride, padding=pad).permute(0, 2, 3, 1)
    assert torch.equal(torch.isfinite(y.float().cpu().reshape(ref.shape)), torch.isfinite(ref))
    grad = st.regions[1][st.P * 4:].view(torch.float32)[:cout * r * r * 8].reshape(cout, r, r, 8)[..., :3].cpu()
    xp = torch.nn.functional.pad(torch.from_numpy(x), (0, 0, pad, pad, pad, pad))
    ho, wo = ref.shape[1:3]
    for i in range(r):
        for j in range(r):
            seen = xp[:, i:i + stride * ho:stride, j:j + stride * wo:stride][:, :ho, :wo]
            assert torch.equal(torch.isfinite(grad[:, i, j]).all(0), torch.isfinite(seen).flatten(0, 2).all(0)), (i, j)


@pytest.mark.parametrize("h,w,cin,cout,r,stride,pad,micro,N,kinds", CASES)
def test_the_cases_reach_the_kernels(h, w, cin, cout, r, stride, pad, micro, N, kinds):
    spec = padded(h, w, cin, cout, r, stride, pad)
    assert (routes.conv_first(spec, micro, False), routes.conv_first(spec, micro * N, True)) == kinds


@pytest.mark.parametrize("spec", [conv(8, 8, 16, 64, 3, 1, 1), conv(8, 8, 8, 12, 3, 1, 1), conv(8, 8, 8, 64, 3, 2, 1), conv(8, 8, 8, 64, 5, 1, 2),
                                  conv(16, 16, 8, 64, 7, 1, 3)])
def test_others_do_not(spec):
    assert routes.conv_first(spec, 300, False) == routes.conv_first(spec, 300, True) == 0
