"""The last stage of expectations and gradients: sums over partial rows, at
the row counts where the number of waves per block changes and with ragged
numbers of terms, observables, parameters and samples, against the oracle
(complex128 states: rounding of float64 sums only)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2512_18995_amd as dq
import workloads as W
from gpu_helpers import DEV, normwise, t64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,batch,nobs,terms", [(1, 3, 2, 1), (6, 5, 3, 7), (10, 1, 1, 40), (11, 2, 9, 3), (16, 1, 2, 33)])
def test_expectation_sums(n, batch, nobs, terms):
    rng = np.random.default_rng(40 + n)
    observables = [W.random_pauli_sum(rng, n, terms) + W.sum_z(n) for _ in range(nobs)]
    c = W.Circuit(n, [W.Gate("ry", (q,), "param", q) for q in range(n)], n)
    plan, obs = dq.Plan(c, "c128"), dq.Observable(n, observables)
    psi = rng.standard_normal((batch, 1 << n)) + 1j * rng.standard_normal((batch, 1 << n))
    psi /= np.linalg.norm(psi, axis=1, keepdims=True)
    got = dq.expval(plan, obs, torch.as_tensor(psi, device=DEV)).cpu().numpy()
    want = np.stack([oracle.expvals(n, psi[b], observables) for b in range(batch)])
    normwise(got, want, 1e-12, 1e-13, "expectations")


@pytest.mark.parametrize("n,batch,layers,per_sample", [(3, 1, 1, False), (3, 70, 1, False), (7, 9, 3, True),
                                                       (9, 2, 4, False), (8, 20, 5, False)])
def test_gradient_sums(n, batch, layers, per_sample):
    """Parameters shared over the batch sum batch x waves rows; a parameter
    read by several gates (here by two layers) sums their chain factors."""
    rng = np.random.default_rng(60 + n + batch)
    gates, P = W.hea_layers(n, layers, ("ry", "rz"), "ring")
    gates = gates + [W.Gate("ry", (q,), "param", q, -0.5) for q in range(n)]
    c = W.Circuit(n, gates, P)
    params, _ = W.random_params(rng, c, batch, per_sample)
    observables = [W.sum_z(n)]
    w = rng.standard_normal((batch, 1))
    plan, obs = dq.Plan(c, "c128"), dq.Observable(n, observables)
    st = plan.state(batch, DEV)
    dq.apply_circuit(plan, st, t64(params))
    got, _ = dq.adjoint_grad(plan, obs, st, t64(params), None, t64(w))
    want, _ = oracle.grad_param_shift(c, params, None, observables, w, batch)
    normwise(got.cpu().numpy(), np.asarray(want).reshape(got.shape), 1e-11, 1e-12, "gradients")


@pytest.mark.parametrize("dtype,tol", [("c64", 1e-5), ("c128", 1e-12)])
@pytest.mark.parametrize("n,batch", [(11, 2), (12, 1), (16, 3), (17, 1)])
def test_one_bit_x_terms(dtype, tol, n, batch):
    """Terms X_h and Y_h times Z strings on every wire: lane bits, register
    bits of the first tile set and of the later, padded ones, more than a set
    holds; beside a group of five terms on one X mask (wide pair kernel)."""
    rng = np.random.default_rng(80 + n)

    def term(h, letter):
        zs = {int(w): "Z" for w in rng.choice(n, 3, replace=False)}
        zs[h] = letter
        return (float(rng.standard_normal()), "".join(zs.get(w, "I") for w in range(n)))

    one = [term(h, "XY"[h % 2]) for h in range(n)] + [term(0, "X")] * 13
    pair = [(0.3 * k + 0.1, "X" + "IZ"[k & 1] + "IZ"[(k >> 1) & 1] + "X" + "IZ"[k >> 2] + "I" * (n - 5)) for k in range(5)]
    observables = [one, pair + W.sum_z(n)]
    plan, obs = dq.Plan(W.Circuit(n, []), dtype), dq.Observable(n, observables)
    psi = rng.standard_normal((batch, 1 << n)) + 1j * rng.standard_normal((batch, 1 << n))
    psi /= np.linalg.norm(psi, axis=1, keepdims=True)
    got = dq.expval(plan, obs, torch.as_tensor(psi, dtype=plan.state(1, "cpu").dtype, device=DEV)).cpu().numpy()
    want = np.stack([oracle.expvals(n, psi[b], observables) for b in range(batch)])
    # the sums of many terms nearly cancel on a random state: the tolerance is
    # relative to the sum of the coefficients that multiply unit amplitudes
    scale = np.array([sum(abs(c) for c, _ in o) for o in observables])
    assert np.all(np.abs(got - want) <= tol * scale), (got, want)
