"""tt_kernel_eigh at the edges of the register tridiagonalisation: orders around
multiples of the 8 rows of a leaf and the 16 columns of a wavefront, the largest that it takes (192) and
the first that goes to the grid kernel, with a leading dimension larger than
the order, a matrix that is already tridiagonal, a diagonal one and one with
zero columns.

Bounds: a backward stable reduction leaves eigenvalue errors and residuals of
about n u |A| (n u = 2e-14 at order 193).
"""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _eigh(A, lda):
    import torch
    from paper_2503_18056_amd import _ffi
    lib = _ffi.load()
    n = A.shape[0]
    pad = np.full((n, lda), np.nan)
    pad[:, :n] = A
    d = torch.as_tensor(pad, device="cuda")
    lam = torch.zeros(n, dtype=torch.float64, device="cuda")
    V = torch.zeros((n, n), dtype=torch.float64, device="cuda")
    ws = torch.zeros(max(int(lib.tt_kernel_eigh_workspace(n)), 256), dtype=torch.uint8, device="cuda")
    kept = C.c_int32()
    st = lib.tt_kernel_eigh(C.c_void_p(d.data_ptr()), n, lda, 0.0, C.c_void_p(lam.data_ptr()),
                            C.c_void_p(V.data_ptr()), n, C.byref(kept), C.c_void_p(ws.data_ptr()),
                            ws.numel(), None)
    assert st == 0, lib.tt_kernel_last_error()
    return lam.cpu().numpy(), V.cpu().numpy()[:, :kept.value], kept.value


def _matrix(kind, n):
    rng = np.random.default_rng(7 * n + len(kind))
    if kind == "dense":
        A = rng.standard_normal((n, n))
        A = A @ A.T
    elif kind == "tridiagonal":
        e = rng.standard_normal(max(n - 1, 0))
        A = np.diag(3.0 + rng.random(n)) + np.diag(e, 1) + np.diag(e, -1)
    elif kind == "diagonal":
        A = np.diag(1.0 + rng.random(n))
    else:   # zero rows and columns in the middle
        A = rng.standard_normal((n, n))
        A[n // 3:2 * n // 3] = 0.0
        A = A @ A.T
    return 0.5 * (A + A.T)


@pytest.mark.parametrize("kind", ["dense", "tridiagonal", "diagonal", "zeros"])
@pytest.mark.parametrize("n", [1, 2, 4, 6, 7, 8, 9, 15, 16, 17, 18, 32, 33, 48, 49, 96, 97, 128, 129, 144, 145,
                               176, 177, 190, 191, 192, 193])
def test_eigh_sizes(kind, n):
    A = _matrix(kind, n)
    lam, V, kept = _eigh(A, n + 3)
    ref = np.linalg.eigvalsh(A)[::-1]
    nrm = max(np.abs(ref).max(), 1e-300)
    bound = 20 * n * 2.0 ** -53
    assert np.abs(lam - ref).max() <= bound * nrm
    assert np.abs(A @ V - V * lam[:kept]).max() <= 4 * bound * nrm
    assert np.abs(V.T @ V - np.eye(kept)).max() <= 4 * bound


def _spectrum(kind, n):
    """Spectra that drive the merges' deflation: runs of equal and of nearly
    equal eigenvalues (rotations), two thirds at rounding level, and none."""
    if kind == "runs":
        return np.repeat(np.linspace(1.0, 2.0, (n + 6) // 7), 7)[:n]
    if kind == "near":
        return 1.0 + np.repeat(np.arange((n + 2) // 3), 3)[:n] / n + 1e-15 * np.arange(n)
    if kind == "noise":
        return np.where(np.arange(n) < n // 3, 10.0 ** (-6.0 * np.arange(n) / n), 1e-18)
    return np.linspace(1.0, 3.0, n)


@pytest.mark.parametrize("kind", ["runs", "near", "noise", "spread"])
@pytest.mark.parametrize("n", [9, 16, 17, 31, 33, 63, 64, 65, 72, 127, 128, 129, 255, 256, 257, 320, 513])
def test_eigh_deflation(kind, n):
    """The merges' edges: one block up to 64 rows, tiles of 64 rows by 32
    columns above, panels of 256 rows, the pole weights' own phase from 256."""
    rng = np.random.default_rng(n)
    Q = np.linalg.qr(rng.standard_normal((n, n)))[0]
    A = (Q * _spectrum(kind, n)) @ Q.T
    A = 0.5 * (A + A.T)
    lam, V, kept = _eigh(A, n)
    ref = np.linalg.eigvalsh(A)[::-1]
    nrm = np.abs(ref).max()
    bound = 20 * n * 2.0 ** -53
    assert np.abs(lam - ref).max() <= bound * nrm
    assert np.abs(A @ V - V * lam[:kept]).max() <= 4 * bound * nrm
    assert np.abs(V.T @ V - np.eye(kept)).max() <= 4 * bound


@pytest.mark.parametrize("kind", ["dense", "zeros"])
@pytest.mark.parametrize("n", [193, 208, 255, 256, 257, 383, 384, 385, 512, 704, 705, 1023])
def test_eigh_grid_orders(kind, n):
    """The reduction over several blocks: 16 rows a block, its column classes."""
    A = _matrix(kind, n)
    lam, V, kept = _eigh(A, n + 1)
    ref = np.linalg.eigvalsh(A)[::-1]
    nrm = np.abs(ref).max()
    bound = 20 * n * 2.0 ** -53
    assert np.abs(lam - ref).max() <= bound * nrm
    assert np.abs(A @ V - V * lam[:kept]).max() <= 4 * bound * nrm
    assert np.abs(V.T @ V - np.eye(kept)).max() <= 4 * bound


@pytest.mark.parametrize("p,q", [(140, 130), (600, 256), (600, 260), (560, 520), (65, 65), (90, 70),
                                 (128, 128), (129, 66), (129, 128), (129, 129), (192, 192), (193, 193),
                                 (256, 256), (257, 257), (384, 300), (385, 385), (513, 70), (520, 513),
                                 (720, 704), (760, 705), (1024, 66)])
def test_svd_large_orders(p, q):
    """The bidiagonalisation's column classes and block counts; Golub-Kahan
    orders 2 q around the staged and the unstaged merges (1024 rows)."""
    import torch
    from paper_2503_18056_amd import _ffi
    lib = _ffi.load()
    rng = np.random.default_rng(q)
    U = np.linalg.qr(rng.standard_normal((p, q)))[0]
    W = np.linalg.qr(rng.standard_normal((q, q)))[0]
    sig = np.linspace(2.0, 1.0, q)
    M = (U * sig) @ W.T
    d = torch.as_tensor(M, device="cuda")
    s = torch.zeros(q, dtype=torch.float64, device="cuda")
    V = torch.zeros((q, q), dtype=torch.float64, device="cuda")
    ws = torch.zeros(int(lib.tt_kernel_svd_workspace(p, q)), dtype=torch.uint8, device="cuda")
    kept = C.c_int32()
    st = lib.tt_kernel_svd(C.c_void_p(d.data_ptr()), p, q, q, C.c_void_p(s.data_ptr()),
                           C.c_void_p(V.data_ptr()), q, C.byref(kept), C.c_void_p(ws.data_ptr()),
                           ws.numel(), None)
    assert st == 0, lib.tt_kernel_last_error()
    assert kept.value == q
    Vh = V.cpu().numpy()
    bound = 40 * q * 2.0 ** -53
    assert np.abs(s.cpu().numpy() - sig).max() <= bound * sig[0]
    assert np.abs(Vh.T @ Vh - np.eye(q)).max() <= 4 * bound
    G = M.T @ M if p > q else M @ M.T    # a square matrix: its left vectors
    assert np.abs(G @ Vh - Vh * sig ** 2).max() <= 16 * bound * sig[0] ** 2


@pytest.mark.parametrize("p,q", [(90, 70), (192, 142), (300, 200)])
def test_svd_wide(p, q):
    """The other orientation (read transposed) gives the same singular values and
    the long side's vectors as M V / sigma."""
    import torch
    from paper_2503_18056_amd import _ffi
    lib = _ffi.load()
    rng = np.random.default_rng(p)
    U = np.linalg.qr(rng.standard_normal((p, q)))[0]
    W = np.linalg.qr(rng.standard_normal((q, q)))[0]
    sig = np.linspace(2.0, 1.0, q)
    M = np.ascontiguousarray(((U * sig) @ W.T).T)    # q x p
    pad = np.full((q, p + 5), np.nan)
    pad[:, :p] = M
    d = torch.as_tensor(pad, device="cuda")
    s = torch.zeros(q, dtype=torch.float64, device="cuda")
    V = torch.zeros((q, q), dtype=torch.float64, device="cuda")
    ws = torch.zeros(int(lib.tt_kernel_svd_workspace(q, p)), dtype=torch.uint8, device="cuda")
    kept = C.c_int32()
    st = lib.tt_kernel_svd(C.c_void_p(d.data_ptr()), q, p, p + 5, C.c_void_p(s.data_ptr()),
                           C.c_void_p(V.data_ptr()), q, C.byref(kept), C.c_void_p(ws.data_ptr()),
                           ws.numel(), None)
    assert st == 0, lib.tt_kernel_last_error()
    bound = 40 * q * 2.0 ** -53
    assert kept.value == q
    assert np.abs(s.cpu().numpy() - sig).max() <= bound * sig[0]
    Vh = V.cpu().numpy()
    assert np.abs(Vh.T @ Vh - np.eye(q)).max() <= 4 * bound
    assert np.abs(M @ (M.T @ Vh) - Vh * sig ** 2).max() <= 16 * bound * sig[0] ** 2
