"""The second rounding of TT_ROUND_TWICE at its full capacity: the state's r1_cap
columns and the source's.  Its Gram's partial tiles are one 32-column group more
than tt_round's where r1_cap is a multiple of 32, and with three transport
blocks (Rusanov without diffusion) few ordinates and many cells they are the
largest user of their buffer.

One step against the oracle at 1e-8, the square root of the unit roundoff, to
which Gram matrices resolve; tiles past their buffer lie in the next Gram.
"""
import numpy as np
import pytest

import workloads as wl
from oracle import Setup, metrics, tt

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("r1,nphi", [(256, 32)])
def test_second_rounding_at_the_rank_cap(r1, nphi):
    from paper_2503_18056_amd import TT_ROUND_TWICE, TTState
    p = wl.small_random(nx=128, ny=128, ntheta=8, nphi=nphi, r1=r1, r2=nphi, seed=77, flux="rusanov", s_plus=0.0,
                        tol=1e-12, rmax=r1)
    st = TTState(p, schedule=TT_ROUND_TWICE, max_steps=2)
    st.step(1)
    (X, Th, Ph), _, _ = tt.run(Setup(p), 1, schedule="twice")
    err = metrics.rel_diff(st.cores(), (X, Th, Ph))
    print(f"ranks gpu={st.ranks()} oracle={(X.shape[1], Ph.shape[0])} err={err:.2e}", flush=True)
    assert st.ranks()[0] == r1
    assert err < 1e-8
