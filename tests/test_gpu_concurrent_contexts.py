"""Contexts that step at the same time, each on its own thread and stream, at live
orders whose reductions wait for their own blocks: as many contexts as tt.h
says fit a GPU.  Every kernel sums in a fixed order, so each must end with the bits that
it ends with alone."""
import threading

import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count,r1", [(4, 60), (4, 102), (2, 110)])
def test_contexts_side_by_side(count, r1):
    """Live orders 5 r1 (+ 1): 301 and 511 (two blocks a CU), 551 (one a CU)."""
    import torch
    from paper_2503_18056_amd import TTState
    states, cores = [], []
    for k in range(count):
        p = wl.small_random(nx=40, ny=40, ntheta=8, nphi=32, r1=r1, r2=12, seed=60 + k, tol=1e-12, rmax=r1)
        states.append(TTState(p, stream=torch.cuda.Stream(), max_steps=64))
        cores.append((p["X0"], p["Th0"], p["Ph0"]))

    def go(k, out):
        states[k].tt_set_cores(*cores[k])
        states[k].step(6)
        out[k] = states[k].cores()

    alone, together = {}, {}
    for k in range(count):
        go(k, alone)
        assert alone[k][0].shape[1] == r1  # at the cap: the order that is meant
    for rep in range(3):
        print("together", count, r1, rep, flush=True)
        together.clear()
        ts = [threading.Thread(target=go, args=(k, together)) for k in range(count)]
        for t in ts:
            t.start()
        for t in ts:
            t.join()
        assert sorted(together) == list(range(count))
        for k in range(count):
            for a, b in zip(alone[k], together[k]):
                assert np.array_equal(a, b)
