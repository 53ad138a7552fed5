"""Helpers shared by the tests: error norms and a stage-level oracle/HIP comparison harness."""
import ctypes as C

import numpy as np


def rel_err(got, ref):
    """max |got - ref| / max |ref|  (the tolerance of the parity bar is stated in this norm)."""
    got = np.asarray(got, dtype=np.float64)
    ref = np.asarray(ref, dtype=np.float64)
    assert got.shape == ref.shape, (got.shape, ref.shape)
    if ref.size == 0:
        return 0.0
    return float(np.max(np.abs(got - ref)) / (np.max(np.abs(ref)) + 1e-30))


def rel_l2(got, ref):
    got = np.asarray(got, dtype=np.float64)
    ref = np.asarray(ref, dtype=np.float64)
    return float(np.linalg.norm(got - ref) / (np.linalg.norm(ref) + 1e-30))


def frac_outside(got, ref, tol):
    """Fraction of elements whose error exceeds tol * max|ref|."""
    got = np.asarray(got, dtype=np.float64)
    ref = np.asarray(ref, dtype=np.float64)
    return float(np.mean(np.abs(got - ref) > tol * (np.max(np.abs(ref)) + 1e-30)))


TOL = {"f32": 1e-4, "bf16": 2e-2}


def call_internal(name, *args):
    """Calls a launcher of the library that its own stages call (the symbol's name) on torch's stream: tensors and None are passed as pointers, the rest as it is."""
    import torch
    from paper_2410_14312_amd import load_library

    f = getattr(load_library(), name)
    f.restype = C.c_int
    assert not any(torch.is_tensor(a) and a.dtype == torch.float64 for a in args), "no launcher takes doubles (the default type of some processes)"
    passed = [C.c_void_p(a.data_ptr()) if torch.is_tensor(a) else C.c_void_p() if a is None else a for a in args]
    assert f(*passed, C.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0, name
