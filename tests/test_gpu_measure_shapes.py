"""Marginal probabilities in every form that the launch chooses between: one
outcome per block (few rows an outcome; many outcomes inside the row and few
blocks), rows by one group of threads and by four; shots by scanning and from
sums formed once per block.  Against the oracle; and the time of the forms
where the choice matters, against a call of the same size."""
import numpy as np
import pytest
import torch

import oracle
import paper_2512_18995_amd as dq
import workloads as W
from gpu_helpers import CT, DEV, normwise

pytestmark = pytest.mark.gpu


def _micros(call):
    call()
    best = np.inf
    for _ in range(7):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(20):
            call()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3 / 20)
    return best


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n,batch,wires", [
    (14, 3, range(5)), (15, 1, range(6)), (19, 1, [4, 0, 2, 1, 3]), (20, 1, range(5)),      # above the row: 1, 2, 32, 64 rows
    (18, 1, range(10, 18)), (18, 1, [17, 9, 13, 8, 16, 10, 15, 11, 12, 14]),                # inside it: few blocks
    (16, 32, range(8, 16)), (17, 40, [16, 12, 3]), (17, 3, [0, 16, 8, 7]),                  # rows shared by four groups
    (20, 4, [5, 11, 6, 10, 7, 9, 8]), (21, 1, range(3, 13)), (2, 300, [1]), (4, 70, [3, 0])])
def test_marginals_of_every_form(dtype, n, batch, wires):
    """Every amplitude is exact in float64, so only the float64 sums of up to 2^20 terms round."""
    rng = np.random.default_rng(n + len(wires))
    plan = dq.Plan(W.Circuit(n, []), dtype)
    psi = torch.as_tensor(rng.standard_normal((batch, 1 << n, 2)), device=DEV)
    st = torch.view_as_complex(psi).to(CT[dtype])
    host = st.cpu().numpy().astype(np.complex128)
    got = dq.probs(plan, st, list(wires)).cpu().numpy()
    for b in range(batch):
        normwise(got[b], oracle.probs(n, host[b], list(wires)), 2.0 ** -40, 0.0, "sample %d" % b)


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("k", [8, 9])
def test_low_wires_take_the_time_of_high_ones(dtype, k):
    """20 qubits, the lowest and the highest wires: 1.4 and 2.3 times apart (7 and 9 where one block read the whole
    state for want of workspace)."""
    n = 20
    plan = dq.Plan(W.Circuit(n, []), dtype)
    st, out = plan.state(1, DEV).normal_(), torch.empty((1, 1 << k), dtype=torch.float64, device=DEV)
    ws = torch.empty(1 << 20, dtype=torch.uint8, device=DEV)
    low = _micros(lambda: dq.probs(plan, st, range(n - k, n), ws=ws, out=out))
    high = _micros(lambda: dq.probs(plan, st, range(k), ws=ws, out=out))
    assert low < 4 * high + 4, (low, high)


@pytest.mark.parametrize("nout,batch,shots", [(16, 5, 300), (17, 5, 300), (64, 1, 513), (64, 3000, 2), (200, 1500, 7),
                                              (1024, 2, 256), (2500, 900, 1), (1, 70, 3)])
def test_shots_of_every_form(nout, batch, shots):
    """Equal outcomes, with uniforms on the sums and above the total, zeros at both ends, a falling and an ended sum."""
    rng = np.random.default_rng(nout + batch)
    p = rng.uniform(0, 1, (batch, nout)) * (rng.uniform(0, 1, (batch, nout)) < 0.7)
    if nout > 16:
        p[:, :2] = p[:, -3:] = 0.0
        p[1 % batch, 7], p[2 % batch, 9] = -0.5, np.nan
    p /= np.maximum(np.nansum(np.abs(p), axis=1, keepdims=True), 1e-300)
    u = rng.uniform(0, 1, (batch, shots))
    k = min(shots, nout)
    u[::2, :k] = np.cumsum(p, axis=1)[::2, :k]
    u[:, -1] = np.where(np.arange(batch) % 3 == 0, 1.5, u[:, -1])
    got = dq.sample(torch.as_tensor(p, device=DEV), torch.as_tensor(u, device=DEV)).cpu().numpy()
    for b in range(batch):
        assert np.array_equal(got[b], oracle.sample(p[b], u[b])), b


@pytest.mark.parametrize("nout", [8, 64])
def test_many_distributions_take_the_time_of_many_shots(nout):
    """60000 shots of as many distributions and of one: within 2 times (14 and 26 when a block formed every sum)."""
    n = 60000
    p = torch.rand((n, nout), dtype=torch.float64, device=DEV)
    u, out = torch.rand((n, 1), dtype=torch.float64, device=DEV), torch.empty((n, 1), dtype=torch.int64, device=DEV)
    many = _micros(lambda: dq.sample(p, u, out=out))
    one = _micros(lambda: dq.sample(p[:1], u.view(1, n), out=out.view(1, n)))
    assert many < 4 * one + 4, (many, one)
