"""Marginal probabilities in every form that the launch chooses between: one
outcome per block (few rows an outcome; many outcomes inside the row and few
blocks), rows by one group of threads and by four, against the oracle; and the
time of the forms where the choice matters, against a call of the same size."""
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
