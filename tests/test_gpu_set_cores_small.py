"""tt_set_cores of cores that fit one staging chunk (131072 entries): in one
transfer, into the Theta_cat or the X' buffer, whichever holds them; or core by
core where neither does.  The bits come back, a smaller state clears the padding
of a larger one, a refused state changes nothing, and a step from set cores gives
the bits of a context that was created with them."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu
NT, NP = 4, 8


def _cores(ns, r1, r2, seed):
    rng = np.random.default_rng(seed)
    return (rng.standard_normal((ns, r1)), rng.standard_normal((r1, NT, r2)), rng.standard_normal((r2, NP)))


# rank caps (r1, r2): Theta_cat holds all; X' does; neither (X fills X' and the
# rest does not fit), below and near a chunk
@pytest.mark.parametrize("nx,ny,r1,r2", [(6, 5, 3, 2), (50, 40, 1, 1), (50, 40, 8, 2), (100, 163, 8, 2),
                                         (64, 64, 31, 3)])
def test_one_transfer(nx, ny, r1, r2):
    from paper_2503_18056_amd import TTError, TTState
    ns = nx * ny
    p = wl.small_random(nx=nx, ny=ny, ntheta=NT, nphi=NP)
    full, low = _cores(ns, r1, r2, 1), _cores(ns, max(1, r1 // 2), 1, 2)
    st = TTState(p, cores=full, r1_cap=r1, r2_cap=r2)
    assert all(np.array_equal(a, b) for a, b in zip(st.tt_get_cores(), full))
    for k in range(3):
        bad = [c.copy() for c in low]
        bad[k].flat[-1] = np.nan
        with pytest.raises(TTError):
            st.tt_set_cores(*bad)
        assert all(np.array_equal(a, b) for a, b in zip(st.tt_get_cores(), full))
    st.tt_set_cores(*low)
    assert all(np.array_equal(a, b) for a, b in zip(st.tt_get_cores(), low))
    st.step(1)
    fresh = TTState(p, cores=low, r1_cap=r1, r2_cap=r2)
    fresh.step(1)
    assert all(np.array_equal(a, b) for a, b in zip(st.tt_get_cores(), fresh.tt_get_cores()))


@pytest.mark.parametrize("extra", [0, 1])
def test_at_one_chunk(extra):
    """A mesh row below and one above a chunk."""
    from paper_2503_18056_amd import TTState
    nx, ny, r1, r2 = 127, 129 - (1 - extra), 8, 2
    p = wl.small_random(nx=nx, ny=ny, ntheta=NT, nphi=NP)
    full = _cores(nx * ny, r1, r2, 4)
    total = sum(c.size for c in full)
    assert (total > 131072) == bool(extra)
    st = TTState(p, cores=full, r1_cap=16, r2_cap=4)
    st.tt_set_cores(*full)
    assert all(np.array_equal(a, b) for a, b in zip(st.tt_get_cores(), full))
