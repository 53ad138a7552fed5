"""The loss of few rows in one workgroup (logits handed out, gradient, mean over the mini-batch's rows) at the edges of its
lane groups and of its range, and one row and one class beyond it.

Reference: fp64 from the fp32 logits that the stage hands out.  The sums are of at most 512 exponentials (a lane adds 8, then a tree) and of
1024 row losses; each fp32 operation adds half a unit of 2^-24, and expf and logf a few: 1e-5 relative to the largest value."""
import numpy as np
import pytest

from workloads.configs import linear, softmax_ce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("classes,micro,N", [(1, 3, 2), (10, 47, 5), (16, 32, 16), (16, 171, 3), (17, 5, 3), (64, 32, 4), (64, 43, 3), (65, 31, 2), (96, 64, 4),
                                             (128, 64, 1), (129, 2, 2), (512, 8, 2), (512, 6, 3), (513, 8, 2), (8, 205, 5)])
def test_loss_of_few_rows(dtype, classes, micro, N):
    import torch
    from paper_2410_14312_amd import Stage

    rng = np.random.default_rng(classes * 1000 + micro)
    M, din = micro * N, 32
    st = Stage([linear(din, classes, False), softmax_ce(classes)], dtype, micro, N, N, 0.1, 0.9, borrow_input=True)
    st.set_params([{"w": rng.standard_normal((classes, din)).astype(np.float32), "b": rng.standard_normal(classes).astype(np.float32)}, {}])
    x = st.prepare_input(rng.standard_normal((M, din)))
    labels = rng.integers(0, classes, M).astype(np.int32)
    ld = torch.from_numpy(labels).to(st.device)
    y = torch.empty(M, classes, dtype=torch.float32, device=st.device)
    losses = torch.zeros(N, dtype=torch.float32, device=st.device)
    for j in range(N):
        r = slice(j * micro, (j + 1) * micro)
        st.forward_micro(j, x[r], y=y[r], labels=ld[r], loss_out=losses[j:j + 1])
    st.backward(list(range(N)))
    torch.cuda.synchronize()
    z = y.cpu().numpy().astype(np.float64)
    ref_z = x.float().cpu().numpy().astype(np.float64) @ st.get_params()[0]["w"].astype(np.float64).T + st.get_params()[0]["b"]
    assert np.abs(z - ref_z).max() < (1e-4 if dtype == "f32" else 2e-2) * np.abs(ref_z).max()
    e = np.exp(z - z.max(1, keepdims=True))
    p = e / e.sum(1, keepdims=True)
    want = -np.log(p[np.arange(M), labels]).reshape(N, micro).mean(1)
    got = losses.cpu().numpy()
    assert np.abs(got - want).max() < 1e-5 * max(1.0, np.abs(want).max())
    g = (p - (np.arange(classes) == labels[:, None])) / M
    gb = st.get_grads()[0]["b"]
    # (bf16: the stored gradient of every row is rounded, 2^-9 each)
    bar = 1e-5 if dtype == "f32" else 2.0 ** -9
    assert np.abs(gb - g.sum(0)).max() <= bar * np.abs(g).sum(0).max() + 1e-9


def test_a_label_out_of_range_gives_a_nan_loss():
    import torch
    from paper_2410_14312_amd import Stage

    st = Stage([linear(8, 10, False), softmax_ce(10)], "f32", 4, 1, 1, 0.1, 0.9)
    st.set_params([{"w": np.ones((10, 8), np.float32), "b": np.zeros(10, np.float32)}, {}])
    loss = torch.zeros(1, dtype=torch.float32, device=st.device)
    st.forward_micro(0, st.prepare_input(np.ones((4, 8))), labels=torch.tensor([0, 9, 10, 1], dtype=torch.int32, device=st.device), loss_out=loss)
    assert torch.isnan(loss).item()
