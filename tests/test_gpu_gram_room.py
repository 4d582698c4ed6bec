"""The wide Gram (more than 384 columns) in less room than its preferred row slices
need: the sizes that tt_kernel_gram_noalloc takes and refuses, workspaces that
hold one slice per 1024 rows (8 to 64), and a context on such a workspace.

Against A^T A in numpy at 1e-12 of the largest entry: the sums of a few thousand
products of order one round at 2^-53 each, whatever the slices."""
import ctypes as C

import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu
TILE = 128 * 128 * 8


def _least(K, n):
    t = (n + 127) // 128
    return min(max(K // 1024, 8), 64) // 8 * 8 * (t * (t + 1) // 2) * TILE


def _ptr(t):
    return C.c_void_p(t.data_ptr())


def _check(G, A):
    ref = A.T @ A
    assert np.abs(G - ref).max() <= 1e-12 * np.abs(ref).max()


@pytest.mark.parametrize("K,n", [(16384, 512), (8192, 641), (8192, 385), (4096, 896), (100, 400)])
def test_noalloc_takes_what_its_scratch_holds(K, n):
    import torch
    from paper_2503_18056_amd import _ffi
    lib = _ffi.load()
    A = np.random.default_rng(n).standard_normal((K, n))
    d = torch.as_tensor(A, device="cuda")
    G = torch.full((n, n), np.nan, dtype=torch.float64, device="cuda")
    st = lib.tt_kernel_gram_noalloc(_ptr(d), K, n, n, _ptr(G), n, None)
    assert st == 0, lib.tt_kernel_last_error()
    _check(G.cpu().numpy(), A)


@pytest.mark.parametrize("K,n", [(65536, 512), (4096, 897), (1, 1025)])
def test_noalloc_refuses_what_it_refused(K, n):
    """(One slice per 1024 rows does not fit the 32 MiB: refused on the host.)"""
    import torch
    from paper_2503_18056_amd import _ffi
    lib = _ffi.load()
    d = torch.zeros(8, dtype=torch.float64, device="cuda")
    assert lib.tt_kernel_gram_noalloc(_ptr(d), K, n, n, _ptr(d), n, None) == _ffi.TT_ERR_INVALID_ARG
    assert b"scratch" in lib.tt_kernel_last_error()


@pytest.mark.parametrize("single", [False, True])
@pytest.mark.parametrize("K,n", [(16384, 512), (8192, 641), (20000, 897)])
def test_gram_in_a_smaller_workspace(K, n, single):
    import torch
    from paper_2503_18056_amd import _ffi
    lib = _ffi.load()
    A = np.random.default_rng(K).standard_normal((K, n))
    d = torch.as_tensor(A, device="cuda")
    if single:
        d = d.float()
        A = d.double().cpu().numpy()
        full, call = int(lib.tt_kernel_gram_f32_workspace(K, n, n)), lib.tt_kernel_gram_f32
    else:
        full, call = int(lib.tt_kernel_gram_workspace(K, n, n)), lib.tt_kernel_gram
    fixed = 256 + ((n + 64) * 4 + 255) // 256 * 256 * single
    least = fixed + _least(K, n)
    assert least <= full
    for nb in sorted({least, least + 12345, (least + full) // 2, full}):
        print(f"K={K} n={n} workspace {nb} of {full}", flush=True)
        ws = torch.zeros(nb + 4096, dtype=torch.uint8, device="cuda")
        ws[nb:] = 77
        G = torch.full((n, n), np.nan, dtype=torch.float64, device="cuda")
        st = call(_ptr(d), K, n, n, _ptr(G), n, _ptr(ws), nb, None)
        assert st == 0, lib.tt_kernel_last_error()
        _check(G.cpu().numpy(), A)
        assert bool((ws[nb:] == 77).all())
    assert call(_ptr(d), K, n, n, _ptr(G), n, _ptr(ws), least - 1, None) == _ffi.TT_ERR_OOM


def test_context_in_a_smaller_workspace(monkeypatch):
    """16384 cells, concatenated rank capacity 641: 32 row slices preferred, 16
    the least."""
    from paper_2503_18056_amd import TTError, TTState, _ffi
    p = wl.small_random(nx=128, ny=128, ntheta=8, nphi=32, r1=40, r2=12, seed=5, tol=1e-6, rmax=128)
    ref = TTState(p, max_steps=4)
    ref.step(2)
    full = ref.workspace.numel()
    lib = _ffi.load()
    least = full - (32 - 16) * 21 * TILE
    for nb in (least, least + 5 * 21 * TILE):
        monkeypatch.setattr(lib, "tt_workspace_bytes", lambda cfg, n, nb=nb: nb)
        st = TTState(p, max_steps=4)
        st.step(2)
        assert st.ranks() == ref.ranks()
        E0, E1 = ref.tt_energy()[0], st.tt_energy()[0]
        assert float((E0 - E1).abs().max()) <= 1e-9 * float(E0.abs().max())
    monkeypatch.setattr(lib, "tt_workspace_bytes", lambda cfg, n: least - 512)
    with pytest.raises(TTError) as e:
        TTState(p, max_steps=4)
    assert e.value.status == _ffi.TT_ERR_OOM
