"""Two-wire diagonal gates of interpreted workgroup passes wherever their bits
lie (lane, register and wave bits of the tile, in both orders): states and
gradients against the oracle, and the time of passes that hold little else
against one-wave passes of the same circuit."""
import numpy as np
import pytest
import torch

import oracle
import paper_2512_18995_amd as dq
import workloads as W
from gpu_helpers import DEV, RTOL, assert_state, normwise, t64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,batch", [(10, 2), (11, 1), (12, 3)])
@pytest.mark.parametrize("op", ["cz", "cp", "rzz", "mixed"])
def test_every_pair_of_wires(op, n, batch):
    rng = np.random.default_rng(n)
    gates, P = [], 0
    for q in range(n):
        gates.append(W.Gate("ry", (q,), "param", P))
        P += 1
    pairs = [(a, b) for a in range(n) for b in range(n) if a != b]
    for k, p in enumerate(rng.permutation(len(pairs))):
        name = op if op != "mixed" else ("cz", "cp", "rzz", "crz", "crx")[k % 5]
        if name == "cz":
            gates.append(W.Gate("cz", pairs[p]))
        else:
            gates.append(W.Gate(name, pairs[p], "param", P))
            P += 1
        if k % 7 == 0:   # on one wire: other register bits are wanted next
            gates.append(W.Gate("rx", (int(rng.integers(n)),), "param", P))
            P += 1
    c = W.Circuit(n, gates, P)
    params, _ = W.random_params(rng, c)
    observables = [W.tfim_open(n), W.random_pauli_sum(rng, n, 3)]
    plan, obs = dq.Plan(c, "c64"), dq.Observable(n, observables)
    assert "wbits=" in plan.describe()
    st = plan.state(batch, DEV)
    dq.apply_circuit(plan, st, t64(params))
    assert_state(st[batch - 1].cpu().numpy(), oracle.state(c, params), "c64", len(gates))
    w = rng.standard_normal((batch, 2))
    g, _ = dq.adjoint_grad(plan, obs, st, t64(params), None, t64(w))
    want, _ = oracle.grad_param_shift(c, params, None, observables, w.sum(0)[None, :], 1, threads=8)
    normwise(g.cpu().numpy(), np.ravel(want), RTOL["c64"], 1e-5, "gradients")


def _micros(call):
    call()
    best = np.inf
    for _ in range(7):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(10):
            call()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 100)
    return best


@pytest.mark.parametrize("op,n", [("cz", 20), ("cp", 12)])
def test_as_fast_as_one_wave_passes(op, n):
    """Forward for CZ (0.92 of their time; 1.44 when every amplitude was multiplied by its sign), adjoint for
    controlled phases (0.87; 1.16 when the gradient term took every amplitude)."""
    gates, P = [], 0
    for _ in range(2):
        for q in range(n):
            gates.append(W.Gate("ry", (q,), "param", P))
            P += 1
        for q in range(n):
            for r in range(q + 1, min(n, q + 7)):
                gates.append(W.Gate(op, (q, r)) if op == "cz" else W.Gate(op, (q, r), "param", P))
                P += op != "cz"
    c = W.Circuit(n, gates, P)
    p, obs = t64(np.random.default_rng(1).uniform(0, 6, P)), dq.Observable(n, [W.tfim_open(n)])
    times = []
    for opt in ({}, {"tile_bits": 5, "adj_tile_bits": 4}):
        plan = dq.Plan(c, "c64", **opt)
        st, ws = plan.state(1, DEV), plan.workspace(1, False, 2, obs, DEV)
        dq.apply_circuit(plan, st, p, None, ws=ws)
        if op == "cz":
            times.append(_micros(lambda: dq.apply_circuit(plan, st, p, None, ws=ws)))
        else:
            w = t64(np.ones((1, 1)))
            times.append(_micros(lambda: dq.adjoint_grad(plan, obs, st, p, None, w, preserve_state=True, ws=ws)))
    assert times[0] < 1.1 * times[1], times
