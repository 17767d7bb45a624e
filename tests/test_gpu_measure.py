"""Marginal probabilities and shots at the edges of their kernels: registers
shorter than, equal to and just beyond a 4 KiB row, wires that all, partly or
never lie inside the row, several rows per block, a state that starts 8 bytes
off a 16-byte boundary; shots around the 2048-outcome chunk and the 256-shot
block, and distributions whose running sums are not monotone."""
import numpy as np
import pytest
import torch

import oracle
import paper_2512_18995_amd as dq
import workloads as W
from gpu_helpers import CT, DEV, normwise

pytestmark = pytest.mark.gpu


def _wire_lists(n):
    low = [n - 1 - b for b in range(min(n, 10))]           # physical bits 0..9
    lists = [[0], [n - 1], low[:9], low[5:8], list(range(min(n, 12)))]
    lists.append([w for w in (n - 8, 0, n - 1, n - 9, n // 2) if 0 <= w < n])
    return [list(dict.fromkeys(ws)) for ws in lists if ws]


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n,batch", [(1, 2), (7, 3), (8, 1), (9, 2), (10, 1), (13, 3), (19, 1)])
def test_marginals(dtype, n, batch):
    """Every amplitude is exact in float64, so only the float64 sums of up to 2^18 terms round
    (complex64 states: the reference reads the rounded amplitudes too)."""
    rng = np.random.default_rng(900 + n)
    plan = dq.Plan(W.Circuit(n, []), dtype)
    psi = rng.standard_normal((batch, 1 << n)) + 1j * rng.standard_normal((batch, 1 << n))
    psi /= np.linalg.norm(psi, axis=1, keepdims=True)
    buf = torch.empty(batch * (1 << n) + 1, dtype=CT[dtype], device=DEV)
    for off in (0, 1):
        st = buf[off:off + batch * (1 << n)].view(batch, 1 << n)
        st.copy_(torch.as_tensor(psi))
        host = st.cpu().numpy()
        for wires in _wire_lists(n):
            got = dq.probs(plan, st, wires).cpu().numpy()
            want = np.stack([oracle.probs(n, host[b].astype(np.complex128), wires) for b in range(batch)])
            normwise(got, want, 2.0 ** -40, 0.0, "marginal %s" % wires)


@pytest.mark.parametrize("nout,shots", [(1, 1), (2, 257), (1023, 256), (2048, 300), (2049, 513), (5000, 40)])
def test_shots(nout, shots):
    rng = np.random.default_rng(nout)
    batch = 3
    p = rng.uniform(0, 1, (batch, nout)) * (rng.uniform(0, 1, (batch, nout)) < 0.7)
    p /= np.maximum(p.sum(1, keepdims=True), 1e-300)
    if nout > 2:
        p[1, 1], p[2, nout // 2] = -0.01, np.nan          # sums that fall, sums that end
    u = rng.uniform(0, 1, (batch, shots))
    k = min(shots, nout)
    u[:, :k] = np.cumsum(p, axis=1)[:, :k]                # on a boundary: the next outcome
    u[:, -1] = 1.5                                        # above the total
    got = dq.sample(torch.as_tensor(p, device=DEV), torch.as_tensor(u, device=DEV)).cpu().numpy()
    for b in range(batch):
        assert np.array_equal(got[b], oracle.sample(p[b], u[b])), b
