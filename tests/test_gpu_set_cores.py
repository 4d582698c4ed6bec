"""tt_set_cores / tt_get_cores round trips: cores larger than one staging chunk
(131072 entries), exactly at it and one past it, ranks below the capacity after
a state at the capacity (the padding is cleared: a second rounding sees none
of the first state), and refused cores, which leave the state as it was.  The
transfers only move values, so they come back to the bit (X rounded to FP32 in
the mixed form).
"""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu

NT, NP = 8, 16


def _cores(ns, r1, r2, seed):
    rng = np.random.default_rng(seed)
    return (rng.standard_normal((ns, r1)), rng.standard_normal((r1, NT, r2)), rng.standard_normal((r2, NP)))


def _same(got, want, mixed):
    X = want[0].astype(np.float32).astype(np.float64) if mixed else want[0]
    return np.array_equal(got[0], X) and np.array_equal(got[1], want[1]) and np.array_equal(got[2], want[2])


# 64 x 64 x 32 is one chunk exactly
@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("nx,ny,r1", [(5, 3, 2), (64, 64, 32), (65, 63, 33), (131, 91, 23)])
def test_round_trip(nx, ny, r1, mixed):
    from paper_2503_18056_amd import TT_FP32_MIXED, TT_FP64, TTError, TTState
    p = wl.small_random(nx=nx, ny=ny, ntheta=NT, nphi=NP)
    r2 = 5
    full, low = _cores(nx * ny, r1, r2, 1), _cores(nx * ny, max(1, r1 // 3), 2, 2)
    st = TTState(p, cores=full, r1_cap=r1, r2_cap=r2, precision=TT_FP32_MIXED if mixed else TT_FP64)
    assert _same(st.tt_get_cores(), full, mixed)
    st.tt_set_cores(*low)
    assert _same(st.tt_get_cores(), low, mixed)
    for k in range(3):
        bad = [c.copy() for c in full]
        bad[k].flat[-1] = [np.nan, np.inf, 1.795e308][k]
        with pytest.raises(TTError):
            st.tt_set_cores(*bad)
        assert _same(st.tt_get_cores(), low, mixed)
    st.tt_set_cores(*full)
    assert _same(st.tt_get_cores(), full, mixed)


def test_state_after_refusal_steps_on():
    """A refused state in between changes no bit of what the steps give."""
    from paper_2503_18056_amd import TTError, TTState
    p = wl.small_random(nx=24, ny=20, ntheta=NT, nphi=NP)
    out = []
    for refuse in (False, True):
        st = TTState(p, r1_cap=20, r2_cap=8, max_steps=4)
        st.tt_step(2)
        if refuse:
            r1, r2 = st.ranks()
            bad = list(_cores(24 * 20, r1, r2, 3))
            bad[2][-1, -1] = np.nan
            with pytest.raises(TTError):
                st.tt_set_cores(*bad)
        st.tt_step(2)
        out.append(st.tt_get_cores())
    assert all(np.array_equal(a, b) for a, b in zip(*out))
