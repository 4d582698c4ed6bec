"""The eigensolvers at live orders below their capacity, as a run has them: block
counts, register classes, LDS strides and vectors a wavefront follow the live
order, in one work area, while orders go down and up; and the number of kept
vectors, which residuals over the kept ones do not see.
"""
import ctypes as C

import numpy as np
import pytest

import workloads as wl
from oracle import Setup, metrics, tt

pytestmark = pytest.mark.gpu


def test_ranks_down_and_up_in_one_context():
    """One context of concatenated rank capacity 641 steps from states of rank
    r1 (three eigensolves of orders 5 r1 + 1, 5 r1 + 1 and 5 r2 + 1 in a batch):
    one block, 16, 32 and 64 blocks, in an order that goes down and up.
    Against the oracle at the bar of a single step, 1e-10."""
    from paper_2503_18056_amd import TTState
    kw = dict(nx=40, ny=40, ntheta=8, nphi=32, tol=1e-3, rmax=128)
    first = wl.small_random(r1=2, r2=2, seed=1, **kw)
    st = TTState(first, r1_cap=128, r2_cap=32, max_steps=64)
    for k, (r1, r2) in enumerate([(128, 30), (20, 8), (39, 12), (52, 12), (103, 14), (28, 9), (128, 32),
                                  (38, 32), (77, 10), (51, 11), (102, 13)]):
        p = wl.small_random(r1=r1, r2=r2, seed=300 + k, **kw)
        for f in ("kappa", "rho", "cv", "T0"):
            p[f] = first[f]
        st.tt_set_cores(p["X0"], p["Th0"], p["Ph0"])
        st.step(1)
        (X, Th, Ph), _, _ = tt.run(Setup(p), 1)
        err = metrics.rel_diff(st.cores(), (X, Th, Ph))
        print(f"r1={r1} r2={r2}: ranks gpu={st.ranks()} oracle={(X.shape[1], Ph.shape[0])} err={err:.2e}", flush=True)
        assert st.ranks() == (X.shape[1], Ph.shape[0])
        assert err < 1e-10


@pytest.mark.parametrize("n", [1, 2, 9, 64, 65, 192, 193, 257, 322, 513, 641, 705])
def test_eigh_keeps_what_is_positive(n):
    """Eigenvalues 1 .. 3, and the same with a third of them negative: every
    positive one is kept, with its vector."""
    import torch
    from paper_2503_18056_amd import _ffi
    lib = _ffi.load()
    for neg in (0, n // 3):
        rng = np.random.default_rng(n + neg)
        Q = np.linalg.qr(rng.standard_normal((n, n)))[0]
        w = np.linspace(1.0, 3.0, n) * np.where(np.arange(n) < neg, -1.0, 1.0)
        A = (Q * w) @ Q.T
        d = torch.as_tensor(0.5 * (A + A.T), device="cuda")
        lam = torch.zeros(n, dtype=torch.float64, device="cuda")
        V = torch.zeros((n, n), dtype=torch.float64, device="cuda")
        ws = torch.zeros(int(lib.tt_kernel_eigh_workspace(n)), dtype=torch.uint8, device="cuda")
        kept = C.c_int32()
        st = lib.tt_kernel_eigh(C.c_void_p(d.data_ptr()), n, n, 0.0, C.c_void_p(lam.data_ptr()),
                                C.c_void_p(V.data_ptr()), n, C.byref(kept), C.c_void_p(ws.data_ptr()),
                                ws.numel(), None)
        assert st == 0, lib.tt_kernel_last_error()
        assert kept.value == n - neg
        v = V.cpu().numpy()[:, :kept.value]
        assert np.abs(v.T @ v - np.eye(kept.value)).max() <= 80 * n * 2.0 ** -53


@pytest.mark.parametrize("p,q", [(1, 1), (9, 4), (144, 63), (100, 100), (129, 66), (200, 193), (560, 520)])
def test_svd_keeps_all_of_a_well_conditioned_matrix(p, q):
    import torch
    from paper_2503_18056_amd import _ffi
    lib = _ffi.load()
    rng = np.random.default_rng(p + q)
    M = np.linalg.qr(rng.standard_normal((p, q)))[0] * np.linspace(1.0, 3.0, q)
    d = torch.as_tensor(M @ np.linalg.qr(rng.standard_normal((q, q)))[0], device="cuda").contiguous()
    sig = torch.zeros(q, dtype=torch.float64, device="cuda")
    V = torch.zeros((q, q), dtype=torch.float64, device="cuda")
    ws = torch.zeros(int(lib.tt_kernel_svd_workspace(p, q)), dtype=torch.uint8, device="cuda")
    kept = C.c_int32()
    st = lib.tt_kernel_svd(C.c_void_p(d.data_ptr()), p, q, q, C.c_void_p(sig.data_ptr()), C.c_void_p(V.data_ptr()),
                           q, C.byref(kept), C.c_void_p(ws.data_ptr()), ws.numel(), None)
    assert st == 0, lib.tt_kernel_last_error()
    assert kept.value == q
    v = V.cpu().numpy()
    assert np.abs(v.T @ v - np.eye(q)).max() <= 80 * q * 2.0 ** -53
    assert np.abs(sig.cpu().numpy() - np.linspace(3.0, 1.0, q) if q > 1 else 0.0).max() <= 60 * q * 2.0 ** -53
