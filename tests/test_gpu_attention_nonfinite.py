"""Infinities and NaN in attention reach what depends on them and nothing else: one element of q, k, v or of the output gradient is
not finite, and every row of the result and of the gradients that does not see its position equals the one of finite data.
(The kernels multiply whole 32 x 32 blocks, so excluded pairs and padded rows meet a probability of zero.)  Where a
non-finite value of v or of the output gradient is seen, it stays in its own feature.

Bound: rows that meet such a value are formed again with fp32 probabilities.  In bf16 with 64 features per head the finite run
rounds them to bf16 (2^-9) before the second product, as it does the stored results: 2^-9 (sum of p |v|) + 2^-9 |o| < 2e-2 of
the largest value.  In fp32 both are sums of at most 300 fp32 products: < 1e-4."""
import numpy as np
import pytest

from tests.util import TOL
from workloads.configs import attention

pytestmark = pytest.mark.gpu

CASES = [
    # (s, d, heads, samples)
    (40, 64, 2, 2),       # 32 features per head: few (batch, head) pairs, the key range split over the waves
    (97, 128, 2, 2),      # 64 features
    (200, 256, 8, 24),    # tiled, 32 features, four and eight waves
    (300, 256, 8, 12),
    (200, 256, 4, 40),    # tiled, 64 features
    (300, 512, 8, 16),
    (33, 48, 3, 1),       # 16 features: the kernels by rows
]


def _run(st, qkv, dout):
    import torch
    o = torch.empty(dout.shape, dtype=st.act_dtype, device=st.device)
    dqkv = torch.empty(qkv.shape, dtype=st.act_dtype, device=st.device)
    st.forward_micro(0, qkv, y=o)
    st.backward([0], dy=dout, dx=dqkv)
    torch.cuda.synchronize()
    return o.double().cpu().numpy(), dqkv.double().cpu().numpy()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("s,d,heads,samples", CASES)
def test_non_finite_values_reach_only_what_sees_them(dtype, s, d, heads, samples):
    import torch
    from paper_2410_14312_amd import Stage
    st = Stage([attention(s, d, heads)], dtype, samples, 1, 1, 0.1, 0.9, borrow_input=True, device="cuda:0")
    gen = torch.Generator(device="cuda").manual_seed(s + d)
    qkv = torch.randn(samples, s, 3 * d, generator=gen, device="cuda").to(st.act_dtype)
    dout = torch.randn(samples, s, d, generator=gen, device="cuda").to(st.act_dtype)
    o0, g0 = _run(st, qkv, dout)
    assert np.isfinite(o0).all() and np.isfinite(g0).all()
    dh = d // heads
    b, h, f = samples - 1, heads - 1, 3

    def same(got, want, keep, what):
        err = np.abs(got[keep] - want[keep])
        assert np.isfinite(got[keep]).all(), what + ": %d of %d values not finite" % ((~np.isfinite(got[keep])).sum(), keep.sum())
        assert err.size == 0 or err.max() <= TOL[dtype] * np.abs(want).max(), what

    for part in ("q", "k", "v", "dout"):
        for t in sorted({5, s // 2, s - 1}):
            for value in (float("inf"), float("nan")):
                what = "%s[%d] = %g" % (part, t, value)
                x, dy = qkv.clone(), dout.clone()
                if part == "dout":
                    dy[b, t, h * dh + f] = value
                else:
                    x[b, t, "qkv".index(part) * d + h * dh + f] = value
                o, g = _run(st, x, dy)
                ko, kg = np.ones(o.shape, bool), np.ones(g.shape, bool)   # what must not change
                cols = lambda i: slice(i * d + h * dh, i * d + (h + 1) * dh)
                if part in ("k", "v"):
                    kg[b, t:, cols(0)] = False         # queries that see position t
                    kg[b, :, cols(1)] = False          # (every key is seen by the last query)
                    if part == "k":
                        ko[b, t:, cols(0)] = False
                        kg[b, :, cols(2)] = False
                    else:
                        ko[b, t:, h * dh + f] = False
                else:
                    kg[b, t, cols(0)] = False
                    kg[b, :t + 1, cols(1)] = False     # keys that query t sees
                    if part == "q":
                        ko[b, t, cols(0)] = False
                        kg[b, :t + 1, cols(2)] = False
                    else:
                        kg[b, :t + 1, 2 * d + h * dh + f] = False
                same(o, o0, ko, what + ": output")
                same(g, g0, kg, what + ": gradient")
                if part == "v":
                    seen = o[b, t:, h * dh + f]
                    assert np.isnan(seen).all() if np.isnan(value) else np.isposinf(seen).all(), what
                if part == "dout":
                    seen = g[b, :t + 1, 2 * d + h * dh + f]
                    assert np.isnan(seen).all() if np.isnan(value) else np.isposinf(seen).all(), what
