"""Which kernel a contraction of a layer runs on, asked of the library's own planning functions (host code, no GPU): tests that
name a kernel check with it that their cases still reach that kernel when the rules change."""
import ctypes as C

from paper_2410_14312_amd import load_library


class _Plan(C.Structure):
    _fields_ = [("bm", C.c_int), ("bn", C.c_int), ("slices", C.c_int), ("kind", C.c_int), ("cost", C.c_double)]


class _Conv(C.Structure):
    _fields_ = [(n, C.c_int) for n in ("B", "H", "W", "Cin", "Ho", "Wo", "Cout", "R", "S", "stride", "pad")]


def _functions():
    lib = load_library()
    plan, small, rows = (getattr(lib, n) for n in ("_ZN4tmps8plan_forElllbii", "_ZN4tmps15small_is_betterEllliRKNS_5Plan2E",
                                                   "_ZN4tmps17conv_rows_variantERKNS_9ConvShapeEliid"))
    persistent = {}   # the rules of the persistent kernel
    for name, result in (("g3_forward_ok", C.c_bool), ("g3_narrow_ok", C.c_bool), ("g3_wgrad_slices", C.c_int), ("g3_long_k_slices", C.c_int)):
        f = persistent[name] = getattr(lib, "_ZN4tmps%d%sElll" % (len(name), name))
        f.restype, f.argtypes = result, [C.c_long, C.c_long, C.c_long]
    plan.restype, plan.argtypes = _Plan, [C.c_long, C.c_long, C.c_long, C.c_bool, C.c_int, C.c_int]
    small.restype, small.argtypes = C.c_bool, [C.c_long, C.c_long, C.c_long, C.c_int, C.POINTER(_Plan)]
    rows.restype, rows.argtypes = C.c_int, [C.POINTER(_Conv), C.c_long, C.c_int, C.c_int, C.c_double]
    return plan, small, rows, persistent


KINDS = ("tiled", "by_k", "async")
DENSE, CONV = 1, 2   # operands that a kernel with asynchronous copies can address: matrices, a convolution's


FORWARD, INPUT, WEIGHT = range(3)


def _route(M, N, K, which, esize, operands):
    plan, small, _, g3 = _functions()
    p = plan(M, N, K, which == WEIGHT, esize, operands)
    if operands == DENSE and esize == 2:   # (the persistent kernel's rules come first)
        if g3["g3_wgrad_slices"](M, N, K) if which == WEIGHT else g3["g3_forward_ok"](M, N, K):
            return "persistent"
        if which == INPUT and g3["g3_long_k_slices"](M, N, K) > 1:
            return "persistent split"
        if (which == INPUT or which == FORWARD and K >= 1024) and g3["g3_narrow_ok"](M, N, K):
            return "persistent narrow"
    if operands == DENSE and small(M, N, K, esize, C.byref(p)):
        return "small"
    if p.kind == 2 and N % 8:
        return "tiled"
    return KINDS[p.kind] + (" split" if p.slices > 1 else "")


def dense_backward_kind(rows, din, dout, dtype):
    """What both gradients of a dense layer run on: 0 two launches, 1 / 2 one of the small / the tiled kernel."""
    f = getattr(load_library(), "_ZN4tmps13backward_kindEllli")
    f.restype, f.argtypes = C.c_int, [C.c_long, C.c_long, C.c_long, C.c_int]
    return f(rows, din, dout, 2 if dtype == "bf16" else 4)


def dense_waits(rows, din, dout, dtype):
    """Whether the weight gradient of a stage's only dense layer waits for the launch at the end of a backward pass."""
    lib = load_library()
    asked, elems = getattr(lib, "_ZN4tmps18dense_wgrad_groupsEilii"), getattr(lib, "_ZN4tmps23dense_wgrad_group_elemsElPA2_Kii")
    asked.restype, elems.restype = C.c_bool, C.c_int64
    return asked(C.c_int(1 if dtype == "bf16" else 0), C.c_long(rows), din, dout) and elems(C.c_long(rows), (C.c_int * 2)(din, dout), 1) >= 0


def dense_routes(sp, dtype, micro, N):
    """(forward, input gradient, weight gradient) of a linear layer whose widths are whole 16-byte chunks, alone in a stage that hands a gradient down."""
    e, rows = 2 if dtype == "bf16" else 4, sp.get("rows", 1)
    din, dout, mb, M = sp["din"], sp["dout"], micro * rows, micro * N * rows
    assert din % (16 // e) == 0 and dout % (16 // e) == 0
    forward, dx, gw = _route(mb, dout, din, FORWARD, e, DENSE), _route(M, din, dout, INPUT, e, DENSE), _route(dout, din, M, WEIGHT, e, DENSE)
    if dense_waits(M, din, dout, dtype):
        return forward, dx, "grouped"
    kind = dense_backward_kind(M, din, dout, dtype)
    return (forward,) + ((dx, gw), ("joint small",) * 2, ("joint tiled",) * 2)[kind]


def pointwise_routes(sp, dtype, micro, N):
    """The same of a 1 x 1 convolution with unit stride (the same contractions over its positions, always one to a launch)."""
    e, rows = 2 if dtype == "bf16" else 4, sp["h"] * sp["w"]
    assert sp["r"] == sp["s"] == sp["stride"] == 1 and sp["pad"] == 0 and sp["cin"] % (16 // e) == 0 and sp["cout"] % (16 // e) == 0
    mb, M, cin, cout = micro * rows, micro * N * rows, sp["cin"], sp["cout"]
    return _route(mb, cout, cin, FORWARD, e, DENSE), _route(M, cin, cout, INPUT, e, DENSE), _route(cout, cin, M, WEIGHT, e, DENSE)


def conv_routes(sp, dtype, micro, N):
    """The same of a convolution with more than one tap (in the natural row order); "rows 443" and the like are the variants
    of the kernel that keeps runs of input rows in LDS."""
    plan, _, rows, _ = _functions()
    e = 2 if dtype == "bf16" else 4
    ho, wo = ((sp[k] + 2 * sp["pad"] - sp[f]) // sp["stride"] + 1 for k, f in (("h", "r"), ("w", "s")))
    taps, cin, cout = sp["r"] * sp["s"], sp["cin"], sp["cout"]
    assert taps > 1 and cin % 8 == 0 and cout % 8 == 0
    out = []
    for B, m, n, c in ((micro, micro * ho * wo, cout, cin), (micro * N, micro * N * sp["h"] * sp["w"], cin, cout)):
        shape = _Conv(B, sp["h"], sp["w"], cin, ho, wo, cout, sp["r"], sp["s"], sp["stride"], sp["pad"])
        v = rows(C.byref(shape), m, n, c, plan(m, n, taps * c, False, 2, CONV).cost / 2400.0) if dtype == "bf16" else 0
        out.append("rows %d" % v if v else _route(m, n, taps * c, FORWARD, e, CONV))
    if dtype == "bf16" and conv_wgrad_rows(sp, micro * N).slices:
        return out[0], out[1], "rows"
    return out[0], out[1], _route(cout, taps * cin, micro * N * ho * wo, WEIGHT, e, CONV)


class _RowsPlan(C.Structure):
    _fields_ = [("slices", C.c_int), ("per_slice", C.c_int)]


def conv_wgrad_plan(sp, samples):
    """What the weight gradient of a convolution runs on where it is not the kernel on runs of rows."""
    ho, wo = ((sp[k] + 2 * sp["pad"] - sp[f]) // sp["stride"] + 1 for k, f in (("h", "r"), ("w", "s")))
    return _functions()[0](sp["cout"], sp["r"] * sp["s"] * sp["cin"], samples * ho * wo, True, 2, CONV)


def conv_first(spec, samples, wgrad):
    """Whether a convolution (a pass of it) runs on the kernels for eight channels: 1 (3 x 3), 2 (7 x 7, stride 2) or 0."""
    f = getattr(load_library(), "_ZN4tmps15conv_first_kindERKNS_9ConvShapeEb")
    f.restype, f.argtypes = C.c_int, [C.POINTER(_Conv), C.c_bool]
    ho, wo = ((spec[k] + 2 * spec["pad"] - spec[r]) // spec["stride"] + 1 for k, r in (("h", "r"), ("w", "s")))
    return f(C.byref(_Conv(samples, spec["h"], spec["w"], spec["cin"], ho, wo, spec["cout"], spec["r"], spec["s"], spec["stride"], spec["pad"])), wgrad)


def conv_wgrad_rows(sp, samples):
    """k-slices and positions of each of a weight gradient on runs of rows (bf16); no slices: it runs on another kernel."""
    f = getattr(load_library(), "_ZN4tmps20conv_wgrad_rows_planERKNS_9ConvShapeERKNS_5Plan2E")
    f.restype, f.argtypes = _RowsPlan, [C.POINTER(_Conv), C.POINTER(_Plan)]
    ho, wo = ((sp[k] + 2 * sp["pad"] - sp[r]) // sp["stride"] + 1 for k, r in (("h", "r"), ("w", "s")))
    shape = _Conv(samples, sp["h"], sp["w"], sp["cin"], ho, wo, sp["cout"], sp["r"], sp["s"], sp["stride"], sp["pad"])
    return f(C.byref(shape), C.byref(conv_wgrad_plan(sp, samples)))
