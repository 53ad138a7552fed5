"""Contractions whose operands have rows (or, where they lie the other way round, k) so far apart that a tile's copies do not reach them with 32-bit offsets, on the
persistent kernel: the instances with an address in each lane.  Which launches those are on the CPU, against the offsets themselves; on the GPU
the layers' functions as a stage calls them (a stage of such a layer with its masters and momentum would hardly fit the card), against products in fp32."""
import ctypes as C

import pytest

from paper_2410_14312_amd import load_library
from tests import routes
from tests.util import call_internal

BF16 = 1


@pytest.mark.parametrize("k_contiguous,rows", [(True, 256), (True, 128), (False, 256), (False, 128)])
def test_launches_with_long_rows_keep_whole_addresses(k_contiguous, rows):
    f = getattr(load_library(), "_ZN4tmps15g3_lane_offsetsEbil")
    f.restype, f.argtypes = C.c_bool, [C.c_bool, C.c_int, C.c_long]
    lines, across = (rows, 64) if k_contiguous else (64, rows)
    limit = (2 ** 31 - across) // (lines - 1) // 8 * 8
    for ld in (64, 768, limit - 8, limit, limit + 8, limit + 16, 2 ** 26, 2 ** 30):
        # (the last chunk's last byte; offsets in a lane are formed modulo 2^32)
        assert f(k_contiguous, rows, ld) == (((lines - 1) * ld + across) * 2 - 1 < 2 ** 32), ld


def _normal(gen, *shape):
    import torch
    return torch.empty(*shape, dtype=torch.bfloat16, device="cuda:0").normal_(generator=gen)


def _product(a, b, step):
    """a [K, m]^T b [K, n] in fp32, `step` of a's columns at a time: yields (first column, product)."""
    for c in range(0, a.shape[1], step):
        yield c, a[:, c:c + step].float().t() @ b.float()


class _Partials(C.Structure):
    _fields_ = [("ws", C.c_void_p), ("later", C.c_void_p)]


class _Job(C.Structure):
    _fields_ = [("dy", C.c_void_p), ("x", C.c_void_p), ("gw", C.c_void_p), ("Din", C.c_int), ("Dout", C.c_int)]


LONG = 2 ** 25 + 2 ** 20 + 8   # the 63rd k after the first lies 2^32 bytes and more behind it


def _check_wgrad(gw, dy, x):
    import torch
    rows, dout, din = dy.shape[0], dy.shape[1], x.shape[1]
    w, b = gw[:dout * din].view(dout, din), gw[dout * din:]
    # sums of `rows` products of size 1 in fp32: each addition rounds by 2^-25 of a sum that stays below 64, once here and once in the reference
    worst = 0.0
    if dout >= din:
        for c, ref in _product(dy, x, 1 << 21):
            worst = max(worst, (w[c:c + ref.shape[0]] - ref).abs().max().item())
    else:
        for c, ref in _product(x, dy, 1 << 21):
            worst = max(worst, (w[:, c:c + ref.shape[0]] - ref.t()).abs().max().item())
    assert worst < rows * 2.0 ** -18, worst
    for c in range(0, dout, 1 << 22):
        assert (b[c:c + (1 << 22)] - dy[:, c:c + (1 << 22)].float().sum(0)).abs().max().item() < rows * 2.0 ** -18


@pytest.mark.gpu
@pytest.mark.parametrize("dout,din", [(LONG, 8), (8, LONG)])
def test_weight_gradient(dout, din):
    import torch
    rows = 64
    assert routes._functions()[3]["g3_wgrad_slices"](dout, din, rows) == 1
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(dout)
    dy, x = _normal(gen, rows, dout), _normal(gen, rows, din)
    gw = torch.zeros(dout * din + dout, dtype=torch.float32, device="cuda:0")
    none = _Partials()
    call_internal("_ZN4tmps11dense_wgradEiPKvS1_PfiiiRKNS_8PartialsEP12ihipStream_t", BF16, dy, x, gw, rows, din, dout, C.byref(none))
    _check_wgrad(gw, dy, x)


GROUPED = [(LONG, 192), (192, LONG), (192, 2 ** 22 + 8)]   # the last one: rows that offsets reach, more columns than the forms of other epilogues take


@pytest.mark.parametrize("dout,din", GROUPED)
def test_the_rule_groups_long_rows(dout, din):
    asked = getattr(load_library(), "_ZN4tmps18dense_wgrad_groupsEilii")
    asked.restype = C.c_bool
    assert asked(BF16, C.c_long(512), din, dout)


@pytest.mark.gpu
@pytest.mark.parametrize("dout,din", GROUPED)
def test_grouped_weight_gradient(dout, din):
    import torch
    rows = 512
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(dout)
    dy, x = _normal(gen, rows, dout), _normal(gen, rows, din)
    gw = torch.zeros(dout * din + dout, dtype=torch.float32, device="cuda:0")
    job = _Job(dy.data_ptr(), x.data_ptr(), gw.data_ptr(), din, dout)
    call_internal("_ZN4tmps17dense_wgrad_groupEiPKNS_13DenseWgradJobEilPflP12ihipStream_t", BF16, C.byref(job), 1, C.c_long(rows), None, C.c_long(0))
    _check_wgrad(gw, dy, x)


@pytest.mark.gpu
def test_long_contractions():
    """Rows of 8.5 million: the 255th after the first lies 2^32 bytes and more behind it.  The forward pass and the input gradient in 256 x 128 tiles, the
    latter in k-slices too."""
    import torch
    M, N, K = 2176, 2048, 2 ** 23 + 2 ** 16 + 64
    g3 = routes._functions()[3]
    assert g3["g3_narrow_ok"](M, N, K) and not g3["g3_forward_ok"](M, N, K)
    slices = g3["g3_long_k_slices"](M, N, K)
    assert slices > 1
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(K)
    a, b = _normal(gen, M, K), _normal(gen, N * K)
    out = torch.empty(M, N, dtype=torch.bfloat16, device="cuda:0")

    def check(right):   # right(k, n): the other operand's rows k .. k + n, [n, N]
        ref = torch.zeros(M, N, dtype=torch.float32, device="cuda:0")
        for k in range(0, K, 1 << 18):
            n = min(1 << 18, K - k)
            ref += a[:, k:k + n].float() @ right(k, n).float()
        # results of one rounding to bf16, 2^-9 of the value; sums of 2^23 products in one order and another, some 2^-24 sqrt(2^23) of a result's size
        err = (out.float() - ref).abs() / (ref.abs() * 2.0 ** -8 + 2.0 ** -10 * K ** 0.5)
        assert err.max().item() < 1.0, err.max().item()

    w = b.view(N, K)
    bias = torch.zeros(N, dtype=torch.float32, device="cuda:0")
    call_internal("_ZN4tmps13dense_forwardEiPKvS1_PKfPviiiiiS1_S4_PfP12ihipStream_t", BF16, a, w, bias, out, M, K, N, 0, 0, None, None, None)
    check(lambda k, n: w[:, k:k + n].t())
    w = b.view(K, N)
    for ws in (None, torch.empty((slices + 1) * M * N, dtype=torch.float32, device="cuda:0")):
        out.zero_()
        call_internal("_ZN4tmps11dense_dgradEiPKvS1_PvS1_iS1_iiiPfP12ihipStream_t", BF16, a, w, out, None, 0, None, M, N, K, ws)
        check(lambda k, n: w[k:k + n])
