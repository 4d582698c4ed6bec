"""NaN and infinity through the eigensolver and the SVD: every call ends, reports
TT_ERR_NUMERIC, and leaves nothing behind that a later call on the same
workspace would see.  The sizes take each route: leaves alone, merges on one
block and over blocks, the register and the multi-block reductions, the Jacobi
SVD and the bidiagonalisation on one and on several blocks.
"""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _ptr(t):
    return C.c_void_p(t.data_ptr())


def _call(lib, torch, what, A, ws):
    d = torch.as_tensor(A, device="cuda")
    m, n = A.shape
    q = min(m, n)
    lam = torch.zeros(q, dtype=torch.float64, device="cuda")
    V = torch.zeros((q, q), dtype=torch.float64, device="cuda")
    kept = C.c_int32()
    if what == "eigh":
        st = lib.tt_kernel_eigh(_ptr(d), n, n, 0.0, _ptr(lam), _ptr(V), n, C.byref(kept), _ptr(ws), ws.numel(), None)
    else:
        st = lib.tt_kernel_svd(_ptr(d), m, n, n, _ptr(lam), _ptr(V), q, C.byref(kept), _ptr(ws), ws.numel(), None)
    return st, lam.cpu().numpy()


@pytest.mark.parametrize("n", [1, 2, 3, 8, 13, 16, 40, 64, 70, 142, 192, 193, 322, 600])
def test_eigh_of_non_finite_matrices(n):
    import torch
    from paper_2503_18056_amd import _ffi
    lib = _ffi.load()
    rng = np.random.default_rng(n)
    A = rng.standard_normal((n, n))
    A = A @ A.T / n + np.eye(n)
    ws = torch.zeros(int(lib.tt_kernel_eigh_workspace(n)), dtype=torch.uint8, device="cuda")
    st, good = _call(lib, torch, "eigh", A, ws)
    assert st == 0
    where = [(n - 1, n - 1), (n // 2, n // 2), (n - 1, 0)]
    for x, (i, j) in [(np.nan, w) for w in where] + ([(np.inf, (n - 1, 0))] if n >= 3 else []):
        print(f"eigh n={n} {x} at {(i, j)}", flush=True)
        B = A.copy()
        B[i, j] = B[j, i] = x
        st, _ = _call(lib, torch, "eigh", B, ws)
        assert st == _ffi.TT_ERR_NUMERIC
    st, _ = _call(lib, torch, "eigh", np.full((n, n), np.nan), ws)
    assert st == _ffi.TT_ERR_NUMERIC
    st, lam = _call(lib, torch, "eigh", A, ws)
    assert st == 0 and np.array_equal(lam, good)


@pytest.mark.parametrize("m,n", [(1, 1), (5, 3), (62, 12), (12, 62), (144, 63), (100, 100), (129, 66), (200, 193)])
def test_svd_of_non_finite_matrices(m, n):
    import torch
    from paper_2503_18056_amd import _ffi
    lib = _ffi.load()
    A = np.random.default_rng(m + n).standard_normal((m, n))
    ws = torch.zeros(int(lib.tt_kernel_svd_workspace(m, n)), dtype=torch.uint8, device="cuda")
    st, good = _call(lib, torch, "svd", A, ws)
    assert st == 0
    for x, (i, j) in [(np.nan, (m - 1, n - 1)), (np.nan, (m // 2, 0)), (np.inf, (0, n // 2))]:
        print(f"svd {m}x{n} {x} at {(i, j)}", flush=True)
        B = A.copy()
        B[i, j] = x
        st, _ = _call(lib, torch, "svd", B, ws)
        if np.isnan(x) or min(m, n) > 1:
            assert st == _ffi.TT_ERR_NUMERIC
    st, sig = _call(lib, torch, "svd", A, ws)
    assert st == 0 and np.array_equal(sig, good)
