"""The vectors of the one-sided Jacobi SVD keep their norms: its rotations'
c^2 + s^2 must not be off one in the mean.

A column of V takes part in at most 10 (q - 1) rotations (sweeps by partners).
With c and s rounded to nearest, each changes its squared norm by at most about
2^-53 at random, so the mean over the q columns of |v_j|^2 - 1 has a standard
deviation of at most sqrt(10 (q - 1) / q) 2^-53, about 3.2 units: the bound is six
of those.  A rotation that is off by half a unit in the mean is off by some 180
at 144 x 63.  The norms are summed in extended precision.
"""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,q", [(96, 32), (142, 36), (36, 142), (144, 63), (220, 60)])
def test_jacobi_vectors_keep_their_norms(p, q):
    import torch
    from paper_2503_18056_amd import _ffi
    lib = _ffi.load()
    k = min(p, q)
    drift = []
    for seed in range(3):
        rng = np.random.default_rng(1000 * p + q + seed)
        M = (10.0 ** (-4.0 * np.arange(p) / p))[:, None] * rng.standard_normal((p, q)) \
            * 10.0 ** (-6.0 * np.arange(q) / q)
        d = torch.as_tensor(M, device="cuda")
        sig = torch.zeros(k, dtype=torch.float64, device="cuda")
        V = torch.zeros((k, k), dtype=torch.float64, device="cuda")
        ws = torch.zeros(int(lib.tt_kernel_svd_workspace(p, q)), dtype=torch.uint8, device="cuda")
        kept = C.c_int32()
        st = lib.tt_kernel_svd(C.c_void_p(d.data_ptr()), p, q, q, C.c_void_p(sig.data_ptr()),
                               C.c_void_p(V.data_ptr()), k, C.byref(kept), C.c_void_p(ws.data_ptr()),
                               ws.numel(), None)
        assert st == 0, lib.tt_kernel_last_error()
        assert kept.value == k
        v = V.cpu().numpy().astype(np.longdouble)
        drift.append(float(np.mean((v * v).sum(axis=0) - 1)) * 2.0 ** 53)
    print("norm drift in units of 2^-53:", drift, flush=True)
    assert np.abs(drift).max() <= 6.0 * np.sqrt(10.0 * (k - 1) / k)
