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


def _batched(dtype, specs):
    plans, obs = [], []
    for n, opt in specs:
        w = W.config(5, n=n, layers=2)
        plans.append(dq.Plan(w.circuit, dtype, **opt))
        obs.append(dq.Observable(n, w.observables))
    return dq.Multi(plans, obs).batched


@pytest.mark.parametrize("adj", [3, 4])
@pytest.mark.parametrize("n", [10, 11, 12, 16])
def test_workgroup_forward_beside_a_one_wave_adjoint_is_batched(n, adj):
    """adj_tile_bits keeps the adjoint in one-wave tiles and leaves the forward its workgroup tiles: each direction
    joins the shared launches in its own form."""
    d = dq.Plan(W.config(5, n=n, layers=2).circuit, "c64", adj_tile_bits=adj).describe().splitlines()
    assert all(("wbits=" in l) == l.startswith("fwd") for l in d if " tile " in l)
    assert _batched("c64", [(n, {"adj_tile_bits": adj})] * 4) == [True] * 4


@pytest.mark.parametrize("dtype,specs", [
    ("c64", [(12, {"tile_bits": 5}), (12, {}), (14, {}), (13, {"tile_bits": 5})]),
    ("c64", [(12, {}), (13, {"tile_bits": 5}), (10, {})]),
    ("c64", [(10, {}), (11, {"tile_bits": 4})]),
    ("c64", [(10, {"jit": True}), (10, {"jit": True}), (10, {})]),
    ("c64", [(10, {"jit": True, "adj_tile_bits": 3}), (10, {"adj_tile_bits": 3})]),
    ("c64", [(12, {"adj_tile_bits": 4}), (13, {"tile_bits": 5}), (14, {})]),
    ("c128", [(10, {"jit": True, "adj_tile_bits": 3}), (11, {})])])
def test_tile_forms_of_one_size_are_batched_together(dtype, specs):
    """One-wave and workgroup tiles of as many register bits, compiled plans of ten qubits included (the shared
    launches interpret them)."""
    assert all(_batched(dtype, specs))


def test_other_sizes_take_the_single_plan_path():
    """The first fused plan sets the size: other one-wave sizes, compiled workgroup tiles of other registers, dense
    blocks and float64 arithmetic stay alone."""
    assert _batched("c64", [(12, {"dense_fuse": 4}), (12, {}), (13, {})]) == [False, True, True]
    assert _batched("c64", [(12, {"tile_bits": 5}), (12, {"tile_bits": 4}), (13, {})]) == [True, False, True]
    assert _batched("c64", [(12, {"jit": True}), (10, {"jit": True})]) == [False, False]
    assert _batched("c64", [(10, {}), (10, {"jit": True, "arith64": True}), (10, {"jit": True})]) == [True, False, True]


@pytest.mark.parametrize("dtype,jit", [("c64", False), ("c64", True), ("c128", True), ("c128", False)])
@pytest.mark.parametrize("n", [8, 10, 20, 31, 32])
def test_candidates_hold_the_default_plan(dtype, jit, n):
    """The tuners can return the plan that a caller gets without options (workgroup tiles from 10 to 31 qubits)."""
    c = W.config(5, n=n, layers=1).circuit
    default = dq.Plan(c, dtype, jit=jit).describe()
    assert any(dq.Plan(c, dtype, tile_bits=o["tile_bits"], dense_fuse=o["dense_fuse"], jit=o["jit"]).describe() == default
               for o in dq.candidate_options(dtype, n, jit))
    if not jit:
        assert n < 9 or any(dq.Plan(c, dtype, **o).describe() == default for o in dq.multi_candidates(dtype))


@pytest.mark.parametrize("unitaries", [0, 1, 3])
def test_steps_without_a_kernel_do_not_share_one(unitaries):
    """Compiled plans of 15 to 17 qubits keep workgroup tiles if two passes share a kernel: sweeps of dense unitaries,
    which have none, do not count as two that do."""
    rng = np.random.default_rng(23)
    c = W.random_circuit(rng, 16, 60, [o for o in W.ALL_OPS if o != "unitary"])
    for k in range(unitaries):
        c.gates.insert(20 * (k + 1), W.Gate("unitary", (k, k + 5, k + 9), matrix=W.random_unitary(rng, 3)))
    steps = [l for l in dq.Plan(c, "c64", jit=True).describe().splitlines() if " tile " in l or " sweep " in l]
    kernels = [l.split(" kernel=")[1].split()[0] for l in steps if " kernel=" in l]
    assert len(kernels) == len(set(kernels)) < len(steps) + (unitaries == 0)
    assert not any("wbits=" in l for l in steps)


def test_a_multi_plan_makes_no_second_plan_of_a_circuit_that_cannot_join():
    """A dense unitary is a sweep of its own in every form: such circuits keep the caller's plan alone."""
    c = W.random_circuit(np.random.default_rng(3), 10, 400, [o for o in W.ALL_OPS if o != "unitary"])
    u = W.Circuit(10, c.gates + [W.Gate("unitary", (1, 4, 7), matrix=W.random_unitary(np.random.default_rng(1), 3))], c.n_params)
    obs = [dq.Observable(10, [W.tfim_open(10)])] * 2
    plans = [dq.Plan(c, "c64"), dq.Plan(u, "c64")]
    assert dq.Multi(plans, obs).batched == [True, False]
    assert _seconds(lambda: dq.Multi(plans, obs)) < 0.5 * _seconds(lambda: dq.Plan(u, "c64"))
