"""Uneven batches whose circuits join the shared launches in different forms
(one-wave tiles, workgroup tiles, compiled plans that the launches interpret,
a direction each) beside some on the single-plan path: every state,
expectation and gradient against the oracle, twice on one workspace."""
import numpy as np
import pytest
import torch

import oracle
import paper_2512_18995_amd as dq
import workloads as W
from gpu_helpers import DEV, RTOL, assert_state, normwise

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,specs,batched", [
    ("c64", [(12, {"adj_tile_bits": 4}), (10, {"adj_tile_bits": 4}), (13, {"adj_tile_bits": 4})], 3),
    ("c64", [(11, {"adj_tile_bits": 3}), (11, {"adj_tile_bits": 3}), (12, {})], 2),
    ("c64", [(12, {"tile_bits": 5}), (12, {}), (9, {}), (13, {"tile_bits": 5}), (14, {})], 4),
    ("c64", [(13, {}), (12, {"tile_bits": 5}), (10, {}), (12, {"adj_tile_bits": 4})], 4),
    ("c64", [(12, {"dense_fuse": 4}), (12, {}), (13, {})], 2),
    ("c64", [(12, {"adj_tile_bits": 4}), (13, {"tile_bits": 5}), (14, {})], 3),
    ("c64", [(10, {"jit": True}), (11, {"tile_bits": 4}), (10, {}), (12, {"jit": True})], 3),
    ("c128", [(10, {"jit": True, "adj_tile_bits": 3}), (11, {}), (12, {})], 3)])
def test_mixed_forms(dtype, specs, batched):
    rng = np.random.default_rng(41)
    ops = [o for o in W.ALL_OPS if o != "unitary"]
    cs = [W.random_circuit(rng, n, 6 * n, ops) for n, _ in specs]
    obs = [[W.tfim_open(c.n), W.random_pauli_sum(rng, c.n, 3)] for c in cs]
    params = [W.random_params(rng, c)[0] for c in cs]
    M = dq.Multi([dq.Plan(c, dtype, **opt) for c, (_, opt) in zip(cs, specs)],
                 [dq.Observable(c.n, o) for c, o in zip(cs, obs)])
    assert sum(M.batched) == batched
    st, ws, p = M.states(DEV), M.workspace(DEV), M.pack_params(params, DEV)
    w = rng.standard_normal(M.nout)
    for _ in range(2):
        M.apply(st, p, ws)
        E, got = M.expval(st, ws).cpu().numpy(), st.cpu()
        g = M.adjoint_grad(st, p, torch.as_tensor(w, device=DEV), ws).cpu().numpy()
        for k, c in enumerate(cs):
            want = oracle.state(c, params[k])
            assert_state(M.state_of(got, k).numpy(), want, dtype, len(c.gates), "circuit %d" % k)
            o = slice(M.out_off[k], M.out_off[k] + 2)
            normwise(E[o], oracle.expvals(c.n, want, obs[k]), RTOL[dtype], 1e-6 if dtype == "c64" else 1e-12, "expval %d" % k)
            ref, _ = oracle.grad_param_shift(c, params[k], None, obs[k], w[o][None, :], 1, threads=8)
            normwise(g[M.param_off[k]:M.param_off[k] + c.n_params], ref, RTOL[dtype], 1e-6 if dtype == "c64" else 1e-12,
                     "gradient %d" % k)
