"""Compiled passes whose tile is shared by the waves of a workgroup: random
circuits of every gate kind and the ring ansatz, in every arithmetic, at the
sizes where the tile's shape changes (the smallest register, a state of one
tile, the first of several tiles, lanes on pinned low bits), with shared and
per-sample angles, against the oracle and the one-wave passes."""
import numpy as np
import pytest
import torch

import oracle
import paper_2512_18995_amd as dq
import workloads as W
from gpu_helpers import CT, DEV, RTOL, assert_state, normwise, rand_state, t64

pytestmark = pytest.mark.gpu
FORMS = [("c64", False), ("c64", True), ("c128", False)]


def _every_gate(rng, n, ngates):
    ops = [o for o in W.ALL_OPS if o != "unitary"] + list(W.TWO_QUBIT_ROT_XY + W.ONE_QUBIT_U3 + W.CONTROLLED_ROT)
    return W.random_circuit(rng, n, ngates, ops, with_data=True)


@pytest.mark.parametrize("dtype,arith64", FORMS)
@pytest.mark.parametrize("n,batch,per_sample", [(10, 3, True), (11, 1, False), (12, 2, False), (13, 2, True),
                                                (15, 2, True)])
def test_random_circuits(dtype, arith64, n, batch, per_sample):
    _random_circuit(dtype, arith64, n, batch, per_sample, True)


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n,batch,per_sample", [(10, 3, True), (11, 70, False), (12, 2, False), (13, 2, True),
                                                (14, 1, False), (16, 2, True)])
def test_random_circuits_interpreted(dtype, n, batch, per_sample):
    """The same passes with their operation list read at run time."""
    _random_circuit(dtype, False, n, batch, per_sample, False)


def test_long_diagonal_runs_interpreted():
    """More one-qubit diagonal gates in a row than one run holds, several on
    each wire, with gradients; then a register of one-qubit gates only."""
    n, rng = 10, np.random.default_rng(5)
    gates = [W.Gate("h", (q,)) for q in range(n)] + [W.Gate("rz", (i % n,), "param", i) for i in range(150)]
    gates += [W.Gate("ry", (q,), "param", 150 + q) for q in range(n)] + W.cnot_ring(n)
    c = W.Circuit(n, gates, 160)
    params, _ = W.random_params(rng, c)
    plan, obs = dq.Plan(c, "c64"), dq.Observable(n, [W.tfim_open(n)])
    assert "wbits=" in plan.describe()
    st = plan.state(1, DEV)
    dq.apply_circuit(plan, st, t64(params))
    assert_state(st[0].cpu().numpy(), oracle.state(c, params), "c64", len(gates))
    g, _ = dq.adjoint_grad(plan, obs, st, t64(params), None, t64(np.ones((1, 1))))
    want, _ = oracle.grad_param_shift(c, params, None, [W.tfim_open(n)], np.ones((1, 1)), 1, threads=8)
    normwise(g.cpu().numpy(), np.ravel(want), RTOL["c64"], 1e-6, "gradients")


def _random_circuit(dtype, arith64, n, batch, per_sample, jit):
    rng = np.random.default_rng(1300 + n)
    c = _every_gate(rng, n, 5 * n)
    params, data = W.random_params(rng, c, batch, per_sample)
    observables = [W.tfim_open(n), W.random_pauli_sum(rng, n, 3)]
    plan, obs = dq.Plan(c, dtype, jit=jit, arith64=arith64), dq.Observable(n, observables)
    if n != 15:   # complex128 interpreted passes keep one-wave tiles
        assert ("wbits=" in plan.describe()) == (jit or dtype == "c64")
    init = rand_state(rng, n)
    st = plan.state(batch, DEV)
    dq.state_init(plan, st, torch.as_tensor(init, dtype=CT[dtype], device=DEV))
    dq.apply_circuit(plan, st, t64(params), t64(data), from_zero=False)
    for b in range(min(batch, 3)):
        assert_state(st[b].cpu().numpy(), oracle.state(c, params, data, b, psi0=init), dtype, len(c.gates), "given state")
    dq.apply_circuit(plan, st, t64(params), t64(data))
    for b in range(min(batch, 3)):
        assert_state(st[b].cpu().numpy(), oracle.state(c, params, data, b), dtype, len(c.gates), "from zero")
    w = rng.standard_normal((batch, 2))
    gp, gd = dq.adjoint_grad(plan, obs, st, t64(params), t64(data), t64(w))
    wp, wd = oracle.grad_param_shift(c, params, data, observables, w, batch, threads=8)
    atol = 1e-5 if dtype == "c64" else 1e-12
    normwise(gp.cpu().numpy().ravel(), np.ravel(wp), RTOL[dtype], atol, "parameter gradients")
    normwise(gd.cpu().numpy().ravel(), np.ravel(wd), RTOL[dtype], atol, "data gradients")


@pytest.mark.parametrize("dtype,arith64,n,jit", [("c64", False, 19, True), ("c64", True, 18, True), ("c128", False, 18, True),
                                                 ("c64", False, 24, True), ("c64", True, 24, True),
                                                 ("c64", False, 19, False), ("c64", False, 21, False),
                                                 ("c64", False, 24, False)])
def test_equals_one_wave_passes(dtype, arith64, n, jit):
    """The ring ansatz at sizes of many tiles (24 qubits: low bits pinned,
    layout searched): the passes of both tile forms apply the same gates."""
    w = W.config(5, n=n, layers=2 if n >= 24 else 4)
    obs = dq.Observable(n, w.observables)
    out = []
    for opt in ({}, {"tile_bits": 5, "adj_tile_bits": 4}):
        plan = dq.Plan(w.circuit, dtype, jit=jit, arith64=arith64, **opt)
        assert ("wbits=" in plan.describe()) == (not opt)
        st = plan.state(1, DEV)
        dq.apply_circuit(plan, st, t64(w.params))
        E = dq.expval(plan, obs, st).cpu().numpy()
        g, _ = dq.adjoint_grad(plan, obs, st, t64(w.params), None, t64(np.ones((1, 1))))
        out.append((E, g.cpu().numpy()))
    normwise(out[0][0], out[1][0], RTOL[dtype], 0.0, "expectation")
    normwise(out[0][1], out[1][1], RTOL[dtype], 0.0, "gradient")
