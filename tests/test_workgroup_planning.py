"""Planning of workgroup tiles (host only)."""
import time

import numpy as np
import pytest

import paper_2512_18995_amd as dq
import workloads as W


def _seconds(make):
    best = np.inf
    for _ in range(3):
        t = time.process_time()
        make()
        best = min(best, time.process_time() - t)
    return best


@pytest.mark.parametrize("jit", [False, True])
def test_planning_time_stays_that_of_one_wave_tiles(jit):
    """The schedule of a workgroup tile's pass is a search; a plan is still made in the time of the plan without
    one: 1.0 to 1.3 times for these circuits (20 times when the search copied its schedule at each of its states)."""
    ops = [o for o in W.ALL_OPS if o != "unitary"]
    for c in (W.random_circuit(np.random.default_rng(17), 12, 600, ops), W.config(5, n=10, layers=60).circuit):
        dq.Plan(c, "c64", jit=jit)
        wide = _seconds(lambda: dq.Plan(c, "c64", jit=jit))
        narrow = _seconds(lambda: dq.Plan(c, "c64", jit=jit, tile_bits=5, adj_tile_bits=4))
        assert wide < 6 * narrow + 0.005, (c.n, wide, narrow)
