"""The loss of rows whose length is no multiple of four: lengths at and around the edges of the kernel's instances, infinities among the logits and labels out of
range, against the definition in 64 bits."""
import numpy as np
import pytest

from workloads.configs import linear, softmax_ce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("C", [2049, 2050, 4095, 4097, 5003, 8191, 8193, 16383, 16385, 32001, 32766, 32769])
def test_against_its_definition(dtype, C):
    """An identity in front, so that the logits are the inputs (bf16 values): rows of the last stage of one linear layer with 32 features, the rest zero."""
    import torch
    from paper_2410_14312_amd import Stage

    rows, M = 37, 2
    rng = np.random.default_rng(C)
    w = np.zeros((C, 32), np.float32)
    at = rng.permutation(C)[:32]
    at[0], at[1], at[2] = 0, C - 1, 2048
    w[at, np.arange(32)] = 1.0
    bias = rng.standard_normal(C).astype(np.float32)
    st = Stage([linear(32, C, False, rows=rows), softmax_ce(C, rows=rows)], dtype, M, 1, 1, 0.5, 0.0, borrow_input=True)
    st.set_params([{"w": w, "b": bias}, {}])
    x = torch.from_numpy(4.0 * rng.standard_normal((M, rows * 32)).astype(np.float32)).to(st.device).to(st.act_dtype)
    labels = torch.from_numpy(rng.integers(0, C, size=(M, rows)).astype(np.int32)).to(st.device)
    labels[0, 0], labels[0, 1], labels[1, 0] = 0, C - 1, 2048
    loss, y = torch.zeros(1, device=st.device, dtype=torch.float32), torch.empty(M, rows * C, device=st.device, dtype=torch.float32)
    st.forward_micro(0, x, y=y, labels=labels, loss_out=loss)
    dx = torch.empty_like(x)
    st.backward([0], dx=dx)
    torch.cuda.synchronize()
    z = y.view(-1, C).double()
    want = torch.nn.functional.cross_entropy(z, labels.view(-1).long())
    assert abs(float(loss) - float(want)) < 2e-6 * abs(float(want))
    p = torch.softmax(z, 1)
    p[torch.arange(p.shape[0]), labels.view(-1).long()] -= 1
    p /= M * rows
    got = torch.from_numpy(np.asarray(st.get_grads()[0]["b"])).to(st.device).double()   # sums of the rounded error signal over the rows
    stored = p.bfloat16().double() if dtype == "bf16" else p
    # in bf16 a value next to a rounding may go the other way: 2^-8 of it, one in some thousand
    assert float(torch.linalg.norm(got - stored.sum(0)) / torch.linalg.norm(stored.sum(0))) < (2e-4 if dtype == "bf16" else 2e-6)


@pytest.mark.parametrize("C", [5003, 16385])
def test_infinities_and_labels_out_of_range(C):
    """An infinite logit or an out-of-range label makes the row's loss NaN, and -inf takes a share of zero."""
    import torch
    from paper_2410_14312_amd import Stage

    def loss_of(bias, label):
        st = Stage([linear(32, C, False), softmax_ce(C)], "bf16", 1, 1, 1, 0.5, 0.0)
        st.set_params([{"w": np.zeros((C, 32), np.float32), "b": bias}, {}])
        loss = torch.zeros(1, device=st.device, dtype=torch.float32)
        st.forward_micro(0, torch.zeros(1, 32, dtype=torch.bfloat16, device=st.device), labels=torch.tensor([[label]], dtype=torch.int32, device=st.device), loss_out=loss)
        torch.cuda.synchronize()
        return float(loss)

    bias = np.zeros(C, np.float32)
    bias[7] = -np.inf
    assert abs(loss_of(bias, 3) - np.log(C - 1)) < 1e-5 and loss_of(bias, 7) == np.inf
    assert np.isnan(loss_of(bias, C)) and np.isnan(loss_of(bias, -1))
    bias[C - 1] = np.inf
    assert np.isnan(loss_of(bias, 3))
