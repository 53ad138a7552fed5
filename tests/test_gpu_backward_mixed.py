"""Both gradients of an fp32 dense layer in one launch on two kernels' tiles: rows and widths at, below and off the edges of 32 x 32 and 64 x 64 tiles.  The
weight gradient is the same bits as without an input gradient; with operands at odd addresses it runs as it did before."""
import ctypes as C

import numpy as np
import pytest

from paper_2410_14312_amd import load_library
from workloads.configs import linear

CASES = [(235, 1000, 1000), (256, 1024, 1024), (225, 996, 1004), (240, 960, 1064), (241, 1000, 1028)]


def takes(rows, din, dout):
    f = getattr(load_library(), "_ZN4tmps20mixed_backward_takesElll")
    f.restype, f.argtypes = C.c_bool, [C.c_long] * 3
    return f(rows, din, dout)


@pytest.mark.parametrize("rows,din,dout", CASES)
def test_the_rule_takes_them(rows, din, dout):
    assert takes(rows, din, dout) and load_library().tmps_dense_gradients_joint(0, C.c_int64(rows), din, dout)


def test_the_rule_leaves_others_alone():
    assert not takes(235, 1000, 1001) and not takes(235, 784, 1000) and not takes(512, 768, 768) and not takes(32, 64, 128)


@pytest.mark.gpu
@pytest.mark.parametrize("odd", [0, 1])
@pytest.mark.parametrize("rows,din,dout", CASES)
def test_both_gradients(rows, din, dout, odd):
    import torch
    from paper_2410_14312_amd import Stage

    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(rows)

    def randn(*shape):
        n = int(np.prod(shape))
        flat = torch.zeros(n + 4, device="cuda:0", dtype=torch.float32)
        flat[odd:odd + n] = torch.randn(n, generator=gen, device="cuda:0", dtype=torch.float32)
        return flat[odd:odd + n].view(shape)

    w, x, dy = randn(dout, din) / din ** 0.5, randn(rows, din), randn(rows, dout)
    got = []
    for down in (True, False):
        st = Stage([linear(din, dout, False)], "f32", rows, 1, 1, 0.1, 0.9, borrow_input=True)
        st.set_params([{"w": w.cpu().numpy(), "b": np.zeros(dout, np.float32)}])
        st.forward_micro(0, x)
        dx = torch.zeros(rows * din + 4, device="cuda:0", dtype=torch.float32)[odd:odd + rows * din].view(rows, din)
        st.backward([0], dy=dy, dx=dx if down else None)
        torch.cuda.synchronize()
        got.append((dx.cpu().numpy(), st.get_grads()[0]))
    (dx, both), (_, alone) = got
    if not odd:
        assert np.array_equal(both["w"], alone["w"]) and np.array_equal(both["b"], alone["b"])
    # sums of products in chains of at most 24 roundings and as many of chains: 2^-24 sqrt(48 / 6), doubled
    for got, want in ((dx, dy.double() @ w.double()), (both["w"], dy.double().t() @ x.double()), (both["b"], dy.double().sum(0))):
        want = want.cpu().numpy()
        assert np.linalg.norm(got - want) < 2 * 2.0 ** -24 * 8 ** 0.5 * np.linalg.norm(want)
