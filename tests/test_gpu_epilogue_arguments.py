"""Every combination of arguments that the dense epilogues take, on each kernel that has instances for some of them: the layers' functions as a stage calls them,
against products in fp32.  Outputs are no whole tiles in either direction; the persistent kernel's have two or three units to a workgroup, so that a unit's stores drain
under the next one's k-tiles and stages are refilled before results, over two k-tiles and over five."""
import ctypes as C
import itertools

import pytest

from paper_2410_14312_amd import load_library
from tests import routes
from tests.util import call_internal

NONE, RELU, GELU = range(3)
SHAPES = [("persistent", 33000, 1000, 128), ("persistent", 33000, 1000, 320), ("persistent narrow", 4200, 1024, 1024), ("async", 1000, 2952, 776), ("by_k", 760, 712, 2056)]
FORWARD = [dict(act=a, bias=b, res=r, second=z) for a, b, r, z in itertools.product((NONE, RELU, GELU), (True, False), (False, True), (False, True))]
INPUT = [dict(mode=m, mask=k, add=a) for m, k in ((RELU, False), (RELU, True), (GELU, True)) for a in ("", "other", "itself")]
AFFINE = [dict(bias=b, again=a, res=r, relu=e) for b, a, r, e in itertools.product((False, True), repeat=4)]


def _form(name, *args):
    lib = load_library()
    f = getattr(lib, {"bias_act": "_ZN4tmps13bias_act_formEibbbl", "conv_affine": "_ZN4tmps16conv_affine_formEbbbbl", "mask": "_ZN4tmps9mask_formEibbl"}[name])
    f.restype = C.c_int
    return f(*[C.c_bool(a) if isinstance(a, bool) else C.c_long(a) if i + 1 == len(args) else a for i, a in enumerate(args)])


@pytest.mark.parametrize("kernel,M,N,K", SHAPES)
def test_shapes_reach_their_kernels(kernel, M, N, K):
    assert [routes._route(M, N, K, which, 2, routes.DENSE) for which in (routes.FORWARD, routes.INPUT)] == [kernel] * 2
    assert kernel != "persistent" or -(-M // 256) * -(-N // 256) > 2 * 256


def test_combinations_are_every_form_and_the_general_epilogue():
    for N in {N for _, _, N, _ in SHAPES}:
        assert {_form("bias_act", c["act"], c["bias"], c["res"], c["second"], N) for c in FORWARD} == {-1, 0, 1, 2, 3}
        assert {_form("mask", c["mode"], c["mask"], c["add"] != "", N) for c in INPUT} == {-1, 0, 1, 2, 3}
        assert {_form("conv_affine", c["bias"], c["again"], c["res"], c["relu"], N) for c in AFFINE} == {-1, 0, 1, 2}
    # rows that a form's offsets do not reach
    assert _form("bias_act", NONE, True, False, False, 2 ** 22) == 0 and _form("bias_act", NONE, True, False, False, 2 ** 22 + 8) == -1
    assert _form("mask", RELU, True, False, 2 ** 22) == 1 and _form("mask", RELU, True, False, 2 ** 22 + 8) == -1
    assert _form("conv_affine", False, False, False, True, 2 ** 22) == 1 and _form("conv_affine", False, False, False, True, 2 ** 22 + 8) == -1


class _Tensors:
    def __init__(self, seed):
        import torch
        self.torch, self.gen = torch, torch.Generator(device="cuda:0")
        self.gen.manual_seed(seed)

    def normal(self, *shape, scale=1.0, dtype=None):
        t = self.torch.empty(*shape, dtype=self.torch.float32, device="cuda:0").normal_(generator=self.gen) * scale
        return t.to(dtype or self.torch.bfloat16)

    def result(self, M, N, dtype=None):
        """[M, N] to be written, in front of a row that is not."""
        return self.torch.full((M + 1, N), float("nan"), device="cuda:0", dtype=dtype or self.torch.bfloat16)

    def check(self, got, ref, what, rel=2.0 ** -8, more=0.0):
        # one rounding to bf16 is 2^-9 of the value; sums of some 2000 products of 1 / sqrt(K) in fp32 are 2^-24 sqrt(K) off and less
        assert self.torch.isnan(got[-1].float()).all(), (what, "written behind the end")
        err = (got[:-1].float() - ref).abs() / (ref.abs() * rel + more + 2.0 ** -16)
        worst = err.max().item()
        assert worst <= 1.0, (what, worst)   # (NaN is not)


def _gelu(v):
    cdf = 0.5 * (1.0 + (v * 0.5 ** 0.5).erf())
    return v * cdf, cdf + v * (-0.5 * v * v).exp() * 0.3989422804014327


@pytest.mark.gpu
@pytest.mark.parametrize("kernel,M,N,K", SHAPES)
def test_forward(kernel, M, N, K):
    import torch
    t = _Tensors(M + K)
    x, w = t.normal(M, K), t.normal(N, K, scale=K ** -0.5)
    bias, res = t.normal(N, dtype=torch.float32), t.normal(M, N)
    product = x.float() @ w.float().t()
    for c in FORWARD:
        for wide in ((False, True) if not c["res"] and not (c["act"] == GELU and c["second"]) else (False,)):   # results in fp32
            out, second = t.result(M, N, torch.float32 if wide else None), t.result(M, N, torch.float32 if wide else None)
            call_internal("_ZN4tmps13dense_forwardEiPKvS1_PKfPviiiiiS1_S4_PfP12ihipStream_t", 1, x, w, bias if c["bias"] else None, out, M, K, N, c["act"], int(wide),
                  res if c["res"] else None, second if c["second"] else None, None)
            v = product + bias if c["bias"] else product
            if c["act"] == RELU:
                v = v.clamp_min(0.0)
            elif c["act"] == GELU:
                v, d = _gelu(v)
            if c["res"]:
                v = v + res.float()
            rel = 2.0 ** -16 if wide else 2.0 ** -8
            t.check(out, v, (c, wide), rel)
            if c["second"]:
                t.check(second, d if c["act"] == GELU else v, (c, wide, "second"), rel)


@pytest.mark.gpu
@pytest.mark.parametrize("kernel,M,N,K", SHAPES)
def test_input_gradient(kernel, M, N, K):
    t = _Tensors(M + K + 1)
    dy, w = t.normal(M, K), t.normal(K, N, scale=K ** -0.5)
    mask, other = t.normal(M, N), t.normal(M, N)
    product = dy.float() @ w.float()
    for c in INPUT:
        out = t.result(M, N)
        if c["add"] == "itself":
            out[:-1] = other
        add = {"": None, "other": other, "itself": out}[c["add"]]
        call_internal("_ZN4tmps11dense_dgradEiPKvS1_PvS1_iS1_iiiPfP12ihipStream_t", 1, dy, w, out, mask if c["mask"] else None, c["mode"], add, M, N, K, None)
        v = product + other.float() if c["add"] else product
        if c["mask"]:
            v = v * mask.float() if c["mode"] == GELU else v * (mask > 0)
        # (a masked sum of cancelling terms is as far off as the sums themselves)
        t.check(out, v, c, more=2.0 ** -16 * 4)


class _Conv(C.Structure):
    _fields_ = [(n, C.c_int) for n in ("B", "H", "W", "Cin", "Ho", "Wo", "Cout", "R", "S", "stride", "pad", "rest_done")]


@pytest.mark.gpu
@pytest.mark.parametrize("kernel,M,N,K", SHAPES)
def test_convolution_with_its_affine_layer(kernel, M, N, K):
    import torch
    t = _Tensors(M + K + 2)
    x, w = t.normal(M, K), t.normal(N, K, scale=K ** -0.5)
    bias, gain, shift, res = t.normal(N, dtype=torch.float32), t.normal(N, dtype=torch.float32), t.normal(N, dtype=torch.float32), t.normal(M, N)
    product = x.float() @ w.float().t()
    shape = _Conv(M // 40, 8, 5, K, 8, 5, N, 1, 1, 1, 0, 0)
    assert shape.B * 40 == M
    for c in AFFINE:
        z, y, again = (t.result(M, N) for _ in range(3))
        call_internal("_ZN4tmps19conv_affine_forwardEiPKvS1_PKfPvS3_S3_S4_S1_S4_iRKNS_9ConvShapeEPfP12ihipStream_t", 1, x, w, bias if c["bias"] else None, z, gain, shift,
              again if c["again"] else None, res if c["res"] else None, y, int(c["relu"]), C.byref(shape), None)
        t.check(z, product + bias if c["bias"] else product, (c, "z"))
        a = (gain * z[:-1].float() + shift).bfloat16().float()   # (from z as it is stored; its rounding may fall to either side: 2^-8 of it)
        v = a + res.float() if c["res"] else a
        if c["relu"]:
            v = v.clamp_min(0.0)
        t.check(y, v, (c, "y"), more=a.abs() * 2.0 ** -7)
        if c["again"]:
            assert torch.equal(again[:-1], y[:-1]) and torch.isnan(again[-1].float()).all(), c
