"""Randomized rounding at the edges of the register Cholesky factor: target ranks
around 16, 32, 64 and 128 (the block counts it is compiled for, and the first that
goes to the global one), against the oracle with the same test matrices.

Bounds: those of the sketch's own tests (both sides orthonormalise the same sketch,
so their projections agree to rounding times the sketch's conditioning): 1e-12
for the tensor, 1e-13 for the factors' orthonormality.
"""
import numpy as np
import pytest

import workloads as wl
from oracle import metrics, rounding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k1,k2", [(1, 1), (2, 2), (15, 15), (16, 16), (17, 3), (31, 4), (32, 5), (33, 6), (63, 7),
                                   (64, 8), (65, 2), (127, 9), (128, 10), (129, 11)])
def test_target_ranks(k1, k2):
    from paper_2503_18056_amd import TTState
    p = wl.small_random(nx=26, ny=23, ntheta=16, nphi=16)
    r1, r2 = 130, 16
    rng = np.random.default_rng(k1)
    X = np.linalg.qr(rng.standard_normal((26 * 23, r1)))[0]
    sc = (0.97 ** np.arange(r1))[:, None, None] * (0.8 ** np.arange(r2))[None, None, :]
    Th = rng.standard_normal((r1, 16, r2)) * sc
    Ph = np.linalg.qr(rng.standard_normal((16, r2)))[0].T
    om = wl.gaussian_test_matrices(16, 16, k1, k2, seed=k1 + 1)
    st = TTState(p, cores=(X, Th, Ph), r1_cap=r1, r2_cap=r2)
    assert st.tt_round_randomized(*om) == (k1, k2)
    Xg, Thg, Phg = st.tt_get_cores()
    assert metrics.rel_diff((Xg, Thg, Phg), rounding.round_randomized(X, Th, Ph, om)) < 1e-12
    T = Thg.reshape(k1 * 16, k2)
    assert np.abs(Xg.T @ Xg - np.eye(k1)).max() < 1e-13
    assert np.abs(T.T @ T - np.eye(k2)).max() < 1e-13
