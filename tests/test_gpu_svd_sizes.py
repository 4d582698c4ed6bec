"""The one-sided Jacobi SVD of M at the edges of its sizes, through
tt_kernel_svd: column blocks (q around multiples of 4), row chunks (p around
multiples of 16 and 64, up to 512), the largest that fit its LDS, both
orientations, against NumPy.

Bounds: singular values carry an absolute error of about q u sigma_1; a
vector's is u sigma_1 / gap; the complement M V / sigma of a vector of M graded on
both sides stays orthogonal to p u sqrt(q) times the spread that its column
scaling leaves (1e-9 here for spreads up to 1e6, where vectors without relative
accuracy give 1e-4).
"""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

U = 2.0 ** -53


def _svd(M):
    import torch
    from paper_2503_18056_amd import _ffi
    lib = _ffi.load()
    a, b = M.shape
    q = min(a, b)
    d = torch.as_tensor(np.ascontiguousarray(M), device="cuda")
    s = torch.zeros(q, dtype=torch.float64, device="cuda")
    V = torch.zeros((a if a <= b else b, q), dtype=torch.float64, device="cuda")
    ws = torch.zeros(max(int(lib.tt_kernel_svd_workspace(a, b)), 256), dtype=torch.uint8, device="cuda")
    kept = C.c_int32()
    st = lib.tt_kernel_svd(C.c_void_p(d.data_ptr()), a, b, b, C.c_void_p(s.data_ptr()),
                           C.c_void_p(V.data_ptr()), q, C.byref(kept), C.c_void_p(ws.data_ptr()),
                           ws.numel(), None)
    assert st == 0, lib.tt_kernel_last_error()
    return s.cpu().numpy(), V.cpu().numpy(), kept.value


SIZES = [(1, 1), (5, 2), (16, 3), (17, 4), (63, 5), (64, 7), (65, 8), (80, 33), (128, 31), (129, 36),
         (192, 64), (193, 40), (208, 64), (224, 64), (225, 63), (253, 40), (257, 40), (281, 40),
         (320, 44), (321, 41), (384, 37), (385, 36), (448, 32), (449, 30), (512, 28), (512, 1)]


@pytest.mark.parametrize("p,q", SIZES)
@pytest.mark.parametrize("tall", [True, False])
def test_jacobi_sizes(p, q, tall):
    rng = np.random.default_rng(1000 * p + q)
    Q = np.linalg.qr(rng.standard_normal((p, q)))[0]
    W = np.linalg.qr(rng.standard_normal((q, q)))[0]
    sig = np.linspace(2.0, 1.0, q)
    B = (Q * sig) @ W.T
    B = B if tall else np.ascontiguousarray(B.T)
    s, V, kept = _svd(B)
    assert kept == q
    assert np.abs(s - sig).max() < 20 * q * U * sig[0]
    assert np.abs(V.T @ V - np.eye(q)).max() < 1e-11
    other = (B @ V if tall else B.T @ V) / s
    assert np.abs(other.T @ other - np.eye(q)).max() < 1e-11
    # each column's largest entry is positive
    assert (V[np.abs(V).argmax(axis=0), np.arange(q)] > 0).all()


@pytest.mark.parametrize("p,q", [(62, 12), (142, 36), (144, 63), (253, 40), (300, 40)])
def test_jacobi_graded(p, q):
    """M = S_A Q S_B, both S falling: the long side's vectors M V / sigma stay
    orthogonal down to the smallest singular value."""
    rng = np.random.default_rng(p)
    Q = np.linalg.qr(rng.standard_normal((p, p)))[0][:, :q]
    M = (10.0 ** (-2.0 * np.arange(p) / p))[:, None] * Q * (10.0 ** (-6.0 * np.arange(q) / q))[None, :]
    s, V, kept = _svd(M)
    assert kept == q
    S = np.linalg.svd(M, compute_uv=False)
    assert np.abs(s - S).max() < 20 * q * U * S[0]
    Un = (M @ V) / s
    assert np.abs(Un.T @ Un - np.eye(q)).max() < 1e-9
