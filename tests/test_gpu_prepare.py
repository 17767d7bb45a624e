"""Gate matrices formed on the device, 64 slots a wave: dense unitaries of one
to five wires as the last slot of a wave, the first of the next and a ragged
tail, per sample, forward and (daggered) in the adjoint, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2512_18995_amd as dq
import workloads as W
from gpu_helpers import DEV, assert_state, normwise, RTOL, t64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("fusion", [True, False])
@pytest.mark.parametrize("first", [0, 60, 63, 64])
def test_unitary_slots(dtype, fusion, first):
    n, batch = 10, 2
    rng = np.random.default_rng(first + 7)
    gates = [W.Gate(("rx", "ry", "rz")[i % 3], (i % n,), "param", i) for i in range(first)]
    for k in (5, 1, 4, 2, 3):
        wires = tuple(int(w) for w in rng.choice(n, k, replace=False))
        gates.append(W.Gate("unitary", wires, matrix=W.random_unitary(rng, k)))
    gates += [W.Gate("u3", (3,), "param", first), W.Gate("swap", (0, 7)), W.Gate("cry", (2, 9), "param", first + 3)]
    c = W.Circuit(n, gates, first + 4)
    params, _ = W.random_params(rng, c, batch, per_sample=True)
    observables = [W.tfim_open(n)]
    plan, obs = dq.Plan(c, dtype, fusion=fusion), dq.Observable(n, observables)
    st = plan.state(batch, DEV)
    dq.apply_circuit(plan, st, t64(params))
    for b in range(batch):
        assert_state(st[b].cpu().numpy(), oracle.state(c, params, None, b), dtype, len(gates), "state %d" % b)
    w = torch.ones((batch, 1), dtype=torch.float64, device=DEV)
    got, _ = dq.adjoint_grad(plan, obs, st, t64(params), None, w)
    want, _ = oracle.grad_param_shift(c, params, None, observables, np.ones((batch, 1)), batch)
    normwise(got.cpu().numpy(), np.asarray(want).reshape(batch, -1), RTOL[dtype], 1e-6 if dtype == "c64" else 1e-12,
             "gradients")
