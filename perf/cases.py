"""Representative workloads of the state-vector engine, as a user's program runs them.

``listed()`` names twelve workloads over the range the engine is used in: two to 28 qubits, one sample to
batches of hundreds, complex64, complex128 and complex64 with float64 arithmetic, interpreted (the default) and
compiled passes, forward only and forward + adjoint, uneven batches, Hessians, measurement.  ``draw(rng)`` gives
one more workload of the same ranges.  ``prepare`` builds the inputs on the GPU, ``run`` makes one pass through
the public entry points, ``exact`` computes the same outputs with plain torch in complex128.
"""
from __future__ import annotations

import functools
import json
import math
from collections import namedtuple

import numpy as np
import torch

import paper_2512_18995_amd as dq

DEV = "cuda:0"

Gate = namedtuple("Gate", "op wires src idx scale matrix")
Circuit = namedtuple("Circuit", "n gates n_params n_data")


# ---------------------------------------------------------------- the workloads
def listed():
    return [
        # curve fitting with the two-wire QResNet: the smallest training step, 16 points, one call of autograd
        dict(name="qresnet_train_n2", kind="train", family="qresnet", n=2, layers=1, batch=16, dtype="c64",
             data_grad=False),
        # the 12-wire QCNN on a batch of encoded images, gradients of weights and of the encoded data
        dict(name="qcnn_train_n12", kind="train", family="qcnn", n=12, layers=1, batch=64, dtype="c64",
             data_grad=True),
        # a small variational eigensolver in double precision: latency of forward + expectation + adjoint
        dict(name="vqe_step_n10_c128", kind="step", rot="yz", ent="ring", obs="z0", n=10, layers=4, batch=1,
             dtype="c128", arith64=False, jit=True, per_sample=False),
        # inference of an encoding circuit over a batch of samples, parameters shared
        dict(name="encode_fwd_n16_b256", kind="forward", n=16, layers=8, batch=256, dtype="c64", jit=True),
        # a batch of independently parameterised circuits under the transverse-field Ising Hamiltonian
        dict(name="tfim_step_n20_b16", kind="step", rot="xyz", ent="czladder", obs="tfim", n=20, layers=12,
             batch=16, dtype="c64", arith64=False, jit=True, per_sample=True),
        # 64 different circuits of 12 to 22 qubits evaluated and differentiated together
        dict(name="uneven_step_64", kind="multi", count=64, nmin=12, nmax=22, lmin=4, lmax=16, terms=8,
             structure=1004),
        # a state beyond every cache, deep enough that its gradient needs float64 arithmetic
        dict(name="vqe_step_n28_arith64", kind="step", rot="yz", ent="ring", obs="zz", n=28, layers=8, batch=1,
             dtype="c64", arith64=True, jit=True, per_sample=False),
        # the quantum Fourier transform of a register that the program holds
        dict(name="qft_n28", kind="qft", n=28, batch=1, dtype="c64", jit=True),
        # all second derivatives of a two-layer circuit (80 parameters)
        dict(name="hessian_n20", kind="hessian", n=20, layers=2, dtype="c64", jit=True),
        # marginal distribution of ten wires of a 27-qubit state, and shots from it
        dict(name="measure_n27", kind="measure", n=27, wires=10, shots=4096, batch=1, dtype="c64"),
        # circuits of dense 2- to 5-qubit unitaries between rotation layers, Pauli-sum expectation
        dict(name="unitary_fwd_n24", kind="unitary", n=24, layers=2, batch=1, dtype="c64", terms=8),
        # Trotterised Ising dynamics in double precision with the default plan, an odd register
        dict(name="trotter_n23_c128", kind="trotter", n=23, steps=6, batch=1, dtype="c128"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))))


def draw(rng):
    """One more workload; sizes are bounded so that none costs more than the 28-qubit gradient step."""
    kind = rng.choice(["train", "train", "step", "step", "forward", "multi", "qft", "hessian", "measure", "unitary",
                       "trotter"])
    if kind == "train":
        family = rng.choice(["qresnet", "qcnn", "encoded", "encoded"])
        n = {"qresnet": 2, "qcnn": 12}.get(family) or rng.randint(3, 14)
        return dict(kind=kind, family=family, n=n, layers=rng.randint(1, 4) if family == "encoded" else 1,
                    batch=_log_int(rng, 1, 300), dtype=rng.choice(["c64", "c64", "c128"]),
                    data_grad=rng.random() < 0.5)
    if kind == "step":
        n = rng.randint(5, 26)
        dtype, arith64 = rng.choice([("c64", False), ("c64", False), ("c64", True), ("c128", False)])
        top = max(1, 1 << max(0, 21 - n))
        return dict(kind=kind, rot=rng.choice(["yz", "xyz"]), ent=rng.choice(["ring", "czladder"]),
                    obs=rng.choice(["zz", "tfim"] + ["z0"] * (n <= 12)), n=n, layers=rng.randint(1, 6),
                    batch=_log_int(rng, 1, min(top, 300)), dtype=dtype, arith64=arith64,
                    jit=arith64 or rng.random() < 0.5, per_sample=rng.random() < 0.5)
    if kind == "forward":
        n = rng.randint(4, 18)
        return dict(kind=kind, n=n, layers=rng.randint(1, 8), batch=_log_int(rng, 1, min(500, 1 << (24 - n))),
                    dtype=rng.choice(["c64", "c64", "c128"]), jit=rng.random() < 0.5)
    if kind == "multi":
        nmin = rng.randint(9, 16)
        return dict(kind=kind, count=_log_int(rng, 4, 64), nmin=nmin, nmax=rng.randint(nmin, 21), lmin=2,
                    lmax=rng.randint(3, 12), terms=rng.randint(4, 8), structure=rng.randint(1, 10 ** 6))
    if kind == "qft":
        return dict(kind=kind, n=rng.randint(10, 27), batch=1, dtype=rng.choice(["c64", "c64", "c128"]),
                    jit=rng.random() < 0.5)
    if kind == "hessian":
        n = rng.randint(4, 17)
        return dict(kind=kind, n=n, layers=rng.randint(1, 2), dtype=rng.choice(["c64", "c128"]),
                    jit=rng.random() < 0.5)
    if kind == "measure":
        n = rng.randint(8, 27)
        return dict(kind=kind, n=n, wires=rng.randint(1, min(12, n)), shots=_log_int(rng, 1, 10000),
                    batch=_log_int(rng, 1, min(200, 1 << (27 - n))), dtype=rng.choice(["c64", "c64", "c128"]))
    if kind == "unitary":
        return dict(kind=kind, n=rng.randint(11, 24), layers=rng.randint(1, 3), batch=rng.randint(1, 3),
                    dtype=rng.choice(["c64", "c64", "c128"]), terms=rng.randint(1, 10))
    n = rng.randint(6, 24)
    return dict(kind="trotter", n=n, steps=rng.randint(1, 8), batch=_log_int(rng, 1, min(100, 1 << (24 - n))),
                dtype=rng.choice(["c64", "c128"]))


# ---------------------------------------------------------------- circuits
def _g(op, wires, src="none", idx=-1, scale=1.0, matrix=None):
    return Gate(op, tuple(wires), src, idx, scale, matrix)


def _ring(n):
    return [_g("cnot", (i, (i + 1) % n)) for i in range(n)]


def _layers(n, layers, rot, ent, gates):
    """Rotation layers (one parameter a gate, kind by kind) with an entangler after each."""
    p = 0
    for _ in range(layers):
        for r in rot:
            for q in range(n):
                gates.append(_g("r" + r, (q,), "param", p))
                p += 1
        gates += _ring(n) if ent == "ring" else [_g("cz", (i, i + 1)) for i in range(n - 1)]
    return p


def _train_circuit(c):
    n, gates, P, D = c["n"], [], 0, 0
    if c["family"] == "qresnet":
        gates = [_g("ry", (0,), "param", 0), _g("u3", (1,), "param", 1), _g("cry", (0, 1), "data", 0),
                 _g("ry", (0,), "param", 4), _g("u3", (1,), "param", 5)]
        return Circuit(2, gates, 8, 1), [[(1.0, "IZ")], [(1.0, "ZZ")]]
    if c["family"] == "encoded":
        gates = [_g("rx", (q,), "data", q) for q in range(n)]
        P = _layers(n, c["layers"], "yz", "ring", gates)
        return Circuit(n, gates, P, n), [[(1.0, _letters(n, {q: "Z"}))] for q in range(min(n, 4))]
    for m in (12, 6, 3):   # encode, convolve neighbours, pool half of the wires away
        for q in range(m):
            gates.append(_g("ry", (q,), "data", D))
            D += 1
        pairs = [(i, i + 1) for i in range(0, m - 1, 2)] if m > 3 else [(0, 1), (1, 2)]
        for pair in pairs:
            for op in ("rxx", "ryy"):
                gates.append(_g(op, pair, "param", P))
                P += 1
        for pair in ([(2 * i + 1, 2 * i) for i in range(m // 2)] if m > 3 else [(1, 0), (2, 0)]):
            gates.append(_g("cry", pair, "param", P))
            P += 1
    return Circuit(n, gates, P, D), [[(1.0, _letters(n, {0: "Z"}))]]


def _letters(n, at):
    return "".join(at.get(w, "I") for w in range(n))


def _observable(kind, n):
    zz = [(1.0, _letters(n, {i: "Z", i + 1: "Z"})) for i in range(n - 1)]
    if kind == "z0":
        return [(1.0, _letters(n, {0: "Z"}))]
    if kind == "sumz":
        return [(1.0, _letters(n, {i: "Z"})) for i in range(n)]
    return zz if kind == "zz" else zz + [(0.5, _letters(n, {i: "X"})) for i in range(n)]


def _pauli_sum(rng, n, terms):
    out = []
    while len(out) < terms:
        s = "".join("IXYZ"[k] for k in rng.integers(0, 4, size=n))
        if s.strip("I"):
            out.append((float(rng.standard_normal()), s))
    return out


def _qft_circuit(n):
    gates = []
    for i in range(n):
        gates.append(_g("h", (i,)))
        gates += [_g("cp", (j + 1, i), scale=math.pi / 2 ** (j - i + 1)) for j in range(i, n - 1)]
    return Circuit(n, gates + [_g("swap", (i, n - 1 - i)) for i in range(n // 2)], 0, 0)


def _trotter_circuit(n, steps):
    """Second-order steps of the periodic Ising chain; parameter 0 is h dt, parameter 1 is J dt."""
    gates = []
    bonds = [(i, i + 1) for i in range(0, n - 1, 2)] + [(i, i + 1) for i in range(1, n - 1, 2)] + [(n - 1, 0)]
    for _ in range(steps):
        gates += [_g("rx", (i,), "param", 0, -1.0) for i in range(n)]
        gates += [_g("rzz", b, "param", 1, -2.0) for b in bonds]
        gates += [_g("rx", (i,), "param", 0, -1.0) for i in range(n)]
    return Circuit(n, gates, 2, 0)


def _random_unitary(rng, k):
    z = rng.standard_normal((1 << k, 1 << k)) + 1j * rng.standard_normal((1 << k, 1 << k))
    q, r = np.linalg.qr(z)
    return q * (np.diag(r) / np.abs(np.diag(r)))[None, :]


def _unitary_circuit(c, seed):
    rng, n, gates, p = np.random.default_rng(seed), c["n"], [], 0
    for layer in range(c["layers"]):
        for q in range(n):
            gates.append(_g("ry", (q,), "param", p))
            p += 1
        order = [int(w) for w in np.random.default_rng(7 + layer).permutation(n)]
        for k in (5, 4, 3, 2):
            block, order = order[:k], order[k:]
            if len(block) == k:
                gates.append(_g("unitary", block, matrix=_random_unitary(rng, k)))
    obs = _observable("tfim", n) + _pauli_sum(np.random.default_rng(11), n, c["terms"])
    return Circuit(n, gates, p, 0), [obs]


def _multi_circuits(c):
    rng, out = np.random.default_rng(c["structure"]), []
    for _ in range(c["count"]):
        n, layers = int(rng.integers(c["nmin"], c["nmax"] + 1)), int(rng.integers(c["lmin"], c["lmax"] + 1))
        gates, p = [], 0
        for _ in range(layers):
            for r in ("ry", "rz"):
                for q in range(n):
                    gates.append(_g(r, (q,), "param", p))
                    p += 1
            perm = rng.permutation(n)
            gates += [_g("cnot", (int(perm[2 * i]), int(perm[2 * i + 1]))) for i in range(n // 2)]
        out.append((Circuit(n, gates, p, 0), [_pauli_sum(rng, n, c["terms"])]))
    return out


def _circuit(c):
    kind, n, gates = c["kind"], c.get("n"), []
    if kind == "train":
        return _train_circuit(c)
    if kind == "step":
        p = _layers(n, c["layers"], c["rot"], c["ent"], gates)
        return Circuit(n, gates, p, 0), [_observable(c["obs"], n)]
    if kind == "forward":
        gates += [_g("rx", (q,), "data", q) for q in range(n)]
        p = _layers(n, c["layers"], "yz", "ring", gates)
        return Circuit(n, gates, p, n), [_observable("sumz", n)]
    if kind == "hessian":
        p = _layers(n, c["layers"], "yz", "ring", gates)
        return Circuit(n, gates, p, 0), [_observable("zz", n)]
    if kind == "trotter":
        return _trotter_circuit(n, c["steps"]), [_observable("tfim", n)]
    if kind == "qft":
        return _qft_circuit(n), None
    return Circuit(n, [], 0, 0), None   # measure: a state that the program holds


# ---------------------------------------------------------------- inputs
@functools.lru_cache(maxsize=1)
def _planned(text):
    """A program plans its circuits once and runs them on new parameters."""
    c = json.loads(text)
    if c["kind"] == "multi":
        both = _multi_circuits(c)
        plans = [dq.Plan(k, "c64") for k, _ in both]
        return dq.Multi(plans, [dq.Observable(k.n, o) for k, o in both]), [k for k, _ in both]
    circuit, obs = _circuit(c)
    plan = dq.Plan(circuit, c["dtype"], jit=c.get("jit", False), arith64=c.get("arith64", False))
    return plan, dq.Observable(circuit.n, obs) if obs else None


def _plan(c):
    return _planned(json.dumps({k: v for k, v in c.items() if k != "name"}, sort_keys=True))


def _angles(gen, *shape, top=2 * math.pi):
    return torch.rand(shape, generator=gen, dtype=torch.float64, device=DEV) * top


def _register(gen, batch, n, dtype):
    """Normalised Gaussian amplitudes: the state of a deep random circuit."""
    real = torch.float32 if dtype == "c64" else torch.float64
    x = torch.randn((batch, 1 << n, 2), generator=gen, dtype=real, device=DEV)
    return torch.view_as_complex(x.mul_(math.sqrt(0.5 / (1 << n))))


def _inputs(c, seed):
    """The numbers of one pass, from the seed alone; shared with exact()."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    kind, s = c["kind"], {}
    if kind == "train":
        circuit, obs = _train_circuit(c)
        s["params"] = _angles(gen, circuit.n_params)
        s["data"] = _angles(gen, c["batch"], circuit.n_data, top=math.pi)
        s["target"] = torch.rand((c["batch"], len(obs)), generator=gen, dtype=torch.float64, device=DEV) * 2 - 1
        if c["dtype"] == "c64":   # a model in single precision holds its weights and data so
            s = {k: v.float() for k, v in s.items()}
    elif kind == "step":
        P = c["n"] * len(c["rot"]) * c["layers"]
        s["params"] = _angles(gen, c["batch"], P) if c["per_sample"] else _angles(gen, P)
    elif kind == "forward":
        s["params"] = _angles(gen, 2 * c["n"] * c["layers"])
        s["data"] = _angles(gen, c["batch"], c["n"], top=math.pi)
    elif kind == "multi":
        s["params"] = [_angles(gen, k.n_params) for k, _ in _multi_circuits(c)]
    elif kind == "hessian":
        s["params"] = _angles(gen, 2 * c["n"] * c["layers"])
    elif kind == "unitary":
        s["params"] = _angles(gen, c["n"] * c["layers"])
    elif kind == "trotter":
        s["params"] = 0.02 + _angles(gen, c["batch"], 2, top=0.2)
    else:
        s["init"] = _register(gen, c["batch"], c["n"], c["dtype"])
        if kind == "measure":
            order = torch.randperm(c["n"], generator=torch.Generator().manual_seed(c["n"] * 31 + c["wires"]))
            s["wires"] = [int(w) for w in order[:c["wires"]]]
            s["uniforms"] = torch.rand((c["batch"], c["shots"]), generator=gen, dtype=torch.float64, device=DEV)
    return s


def prepare(case, seed):
    c, s = case, _inputs(case, seed)
    kind = c["kind"]
    s["kind"], s["dtype"] = kind, c.get("dtype", "c64")
    if kind == "unitary":   # the matrices are this program's weights
        circuit, obs = _unitary_circuit(c, seed)
        s["plan"], s["obs"] = dq.Plan(circuit, c["dtype"]), dq.Observable(c["n"], obs)
    elif kind == "multi":
        s["multi"], _ = _plan(c)
        m = s["multi"]
        s["params"] = m.pack_params(s["params"], DEV)
        s["state"], s["ws"] = m.states(DEV), m.workspace(DEV)
        s["weights"] = torch.ones(m.nout, dtype=torch.float64, device=DEV)
        return s
    else:
        s["plan"], s["obs"] = _plan(c)
    plan, obs, B = s["plan"], s["obs"], c.get("batch", 1)
    if kind == "train":
        s["data_grad"], s["batch"] = c["data_grad"], B
    elif kind in ("step", "forward", "unitary", "trotter"):
        s["state"] = plan.state(B, DEV)
        per_sample = s["params"].dim() == 2 or "data" in s
        s["ws"] = plan.workspace(B, per_sample, 1 if kind == "step" else 0, obs, DEV)
        s["weights"] = torch.ones((B, obs.nobs), dtype=torch.float64, device=DEV)
    elif kind == "qft":
        s["state"], s["ws"] = plan.state(B, DEV), plan.workspace(B, False, 0, None, DEV)
    return s


# ---------------------------------------------------------------- one pass
def run(s):
    kind, plan, obs = s["kind"], s.get("plan"), s.get("obs")
    if kind == "train":
        p = s["params"].detach().requires_grad_()
        d = s["data"].detach().requires_grad_(s["data_grad"])
        E = dq.expectation(plan, obs, p, d, batch=s["batch"])
        ((E - s["target"]) ** 2).mean().backward()
        return [E.detach().to(p.dtype), p.grad] + ([d.grad] if s["data_grad"] else [])
    # a complex64 program goes on in single precision with what it gets
    real = torch.float32 if s["dtype"] == "c64" else torch.float64
    if kind == "step":
        dq.apply_circuit(plan, s["state"], s["params"], ws=s["ws"])
        E = dq.expval(plan, obs, s["state"], ws=s["ws"])
        g, _ = dq.adjoint_grad(plan, obs, s["state"], s["params"], None, s["weights"], ws=s["ws"])
        return [E.to(real), g.to(real)]
    if kind in ("forward", "unitary", "trotter"):
        dq.apply_circuit(plan, s["state"], s["params"], s.get("data"), ws=s["ws"])
        return [dq.expval(plan, obs, s["state"], ws=s["ws"]).to(real), s["state"]]
    if kind == "multi":
        m = s["multi"]
        m.apply(s["state"], s["params"], s["ws"])
        E = m.expval(s["state"], s["ws"])
        return [E.to(real), m.adjoint_grad(s["state"], s["params"], s["weights"], s["ws"]).to(real)]
    if kind == "qft":
        dq.state_init(plan, s["state"], s["init"])
        return [dq.apply_circuit(plan, s["state"], from_zero=False, ws=s["ws"])]
    if kind == "hessian":
        return [dq.hessian(plan, obs, s["params"]).to(real)]
    p = dq.probs(plan, s["init"], s["wires"])
    return [p, dq.sample(p, s["uniforms"])]


# ---------------------------------------------------------------- what a pass cannot do without
def _gate_flops(circuit):
    """Real operations per amplitude of one forward sweep of the circuit."""
    each = {"h": 6, "rx": 6, "ry": 6, "rz": 6, "u3": 14, "cp": 1.5, "rzz": 6, "rxx": 6, "ryy": 6, "crx": 3, "cry": 3,
            "crz": 3, "unitary": 0}
    return sum(8 * (1 << len(g.wires)) - 2 if g.op == "unitary" else each.get(g.op, 0) for g in circuit.gates)


def work(case):
    """Bytes: what the caller hands over and gets back, and where a gradient follows the state written once and
    read once.  Operations: every gate once on the state, in a gradient also twice on the way back with the
    generator's inner product; measurements one read of the state."""
    c, kind = case, case["kind"]
    if kind == "multi":
        by = fl = 0.0
        for k, obs in _multi_circuits(c):
            amps = 2.0 ** k.n
            by += 2 * 8 * amps + 16 * k.n_params
            fl += amps * (3 * _gate_flops(k) + 3 * k.n_params + 8 * len(obs[0]))
        return {"bytes": by, "flops": fl}
    amp = 16 if c["dtype"] == "c128" else 8
    B = c.get("batch", 1)
    amps = B * 2.0 ** c["n"]
    if kind == "measure":
        return {"bytes": amps * amp + 8 * B * (2 ** c["wires"] + 2 * c["shots"]), "flops": 4 * amps}
    circuit, obs = _unitary_circuit(c, 0) if kind == "unitary" else _circuit(c)
    fwd = _gate_flops(circuit)
    terms = sum(len(o) for o in obs) if obs else 0
    if kind == "qft":
        return {"bytes": 2 * amps * amp, "flops": amps * fwd}
    if kind in ("train", "step"):
        g = circuit.n_params + (circuit.n_data if c.get("data_grad") else 0)
        return {"bytes": 2 * amps * amp + 16.0 * g, "flops": amps * (3 * fwd + 3 * g + 8 * terms)}
    if kind == "hessian":
        P = circuit.n_params   # a forward and a reverse sweep of two states for every parameter
        return {"bytes": 8.0 * P * (P + 1), "flops": 2 * P * amps * (3 * fwd + 3 * P)}
    return {"bytes": amps * amp + 8.0 * (circuit.n_params + B * circuit.n_data), "flops": amps * (fwd + 8 * terms)}


# ---------------------------------------------------------------- the same in complex128, with torch alone
_X = torch.tensor([[0, 1], [1, 0]], dtype=torch.complex128)
_Y = torch.tensor([[0, -1j], [1j, 0]], dtype=torch.complex128)
_Z = torch.tensor([[1, 0], [0, -1]], dtype=torch.complex128)
_PAULI = {"x": _X, "y": _Y, "z": _Z}


def _generator(op):
    """G with U(t) = exp(-i t G / 2)."""
    if op in ("rx", "ry", "rz"):
        return _PAULI[op[1]]
    if op in ("rxx", "ryy", "rzz"):
        return torch.kron(_PAULI[op[1]], _PAULI[op[1]])
    if op in ("crx", "cry", "crz"):
        return torch.kron(torch.diag(torch.tensor([0, 1], dtype=torch.complex128)), _PAULI[op[2]])
    if op == "cp":
        return torch.diag(torch.tensor([0, 0, 0, -2], dtype=torch.complex128))
    return torch.diag(torch.tensor([0, -2], dtype=torch.complex128))   # "p", the phase gate diag(1, e^it)


def _simple(gates):
    """U3(a, b, c) as P(b) RY(a) P(c); every other gate as it is."""
    for g in gates:
        if g.op == "u3":
            yield Gate("p", g.wires, g.src, g.idx + 2, g.scale, None)
            yield Gate("ry", g.wires, g.src, g.idx, g.scale, None)
            yield Gate("p", g.wires, g.src, g.idx + 1, g.scale, None)
        else:
            yield g


def _matrix(g, t):
    """[T, d, d] matrices of gate g at the angles t [T]."""
    if g.op == "unitary":
        return torch.as_tensor(g.matrix, dtype=torch.complex128, device=DEV)[None]
    if g.op in ("h", "cnot", "cz", "swap"):
        m = {"h": [[math.sqrt(0.5), math.sqrt(0.5)], [math.sqrt(0.5), -math.sqrt(0.5)]],
             "cnot": [[1, 0, 0, 0], [0, 1, 0, 0], [0, 0, 0, 1], [0, 0, 1, 0]],
             "cz": [[1, 0, 0, 0], [0, 1, 0, 0], [0, 0, 1, 0], [0, 0, 0, -1]],
             "swap": [[1, 0, 0, 0], [0, 0, 1, 0], [0, 1, 0, 0], [0, 0, 0, 1]]}[g.op]
        return torch.tensor(m, dtype=torch.complex128, device=DEV)[None]
    G = _generator(g.op).to(DEV)
    if not bool((G - torch.diag(torch.diagonal(G))).any()):
        return torch.diag_embed(torch.exp(-0.5j * t[:, None] * torch.diagonal(G)[None]))
    P = G @ G   # the projector on which G squares to one
    one = torch.eye(G.shape[0], dtype=torch.complex128, device=DEV)
    c, s = torch.cos(t / 2).to(torch.complex128), torch.sin(t / 2).to(torch.complex128)
    return one[None] + (c - 1)[:, None, None] * P[None] - 1j * s[:, None, None] * G[None]


@functools.lru_cache(maxsize=None)
def _shape(op, generator=False):
    """Which entries of an operation's matrix are not zero, and which diagonal ones are one."""
    if op in _PAULI:
        m = _PAULI[op]
    elif generator:
        m = _generator(op)
    else:
        m = _matrix(Gate(op, (), "none", -1, 1.0, None), torch.full((1,), 0.7, dtype=torch.float64, device=DEV))[0].cpu()
    return (m.abs() > 0).tolist(), (m.diagonal() == 1).tolist()


def _apply(psi, n, wires, m, shape_of=None):
    """m [T, d, d] (T = 1 or the batch) on the wires of psi [B, 2^n]; returns the new state (psi is reused).
    shape_of: the matrix's _shape, for one and two wires."""
    B, k, d = psi.shape[0], len(wires), 1 << len(wires)
    order = sorted(range(k), key=lambda i: wires[i])
    shape, at = [B], 0
    for i in order:
        shape += [1 << (wires[i] - at), 2]
        at = wires[i] + 1
    v = psi.view(shape + [1 << (n - at)])
    place = {i: 2 + 2 * j for j, i in enumerate(order)}   # axis of listed wire i
    if shape_of is None:
        front = [place[i] for i in range(k)]
        rest = [a for a in range(1, v.dim()) if a not in front]
        x = v.permute([0] + front + rest)
        y = torch.matmul(m, x.reshape(B, d, -1)).reshape(x.shape)
        back = [0] * v.dim()
        for a, b in enumerate([0] + front + rest):
            back[b] = a
        return y.permute(back).reshape(B, -1)

    def part(r):
        w = v
        for a, bit in sorted(((place[i], (r >> (k - 1 - i)) & 1) for i in range(k)), reverse=True):
            w = w.select(a, bit)
        return w

    some, unit = shape_of
    new = {}
    for r in range(d):
        cols = [c for c in range(d) if some[r][c]]
        if cols == [r]:
            if not unit[r]:
                w = part(r)
                w.mul_(m[:, r, r].view([-1] + [1] * (w.dim() - 1)))
            continue
        w = None
        for c in cols:
            x = part(c)
            e = m[:, r, c].reshape([-1] + [1] * (x.dim() - 1))
            w = x * e if w is None else w.addcmul_(x, e.expand_as(x))
        new[r] = w
    for r, w in new.items():
        part(r).copy_(w) if w is not None else part(r).zero_()
    return psi


def _pauli(psi, n, letters):
    out = psi.clone()
    for w, l in enumerate(letters):
        if l != "I":
            out = _apply(out, n, (w,), _PAULI[l.lower()].to(DEV)[None], _shape(l.lower()))
    return out


def _vdot(a, b):
    """Row-wise inner products, summed in pieces that stay small beside the states."""
    out = torch.zeros(a.shape[0], dtype=torch.complex128, device=DEV)
    step = 1 << 24
    for i in range(0, a.shape[1], step):
        out += (a[:, i:i + step].conj() * b[:, i:i + step]).sum(1)
    return out


def _observe(psi, n, obs):
    """Expectations [B, nobs]; Z strings from the probabilities."""
    prob = torch.view_as_real(psi).square().sum(-1)
    cols = []
    for o in obs:
        E = torch.zeros(psi.shape[0], dtype=torch.float64, device=DEV)
        for coef, letters in o:
            if set(letters) <= {"I", "Z"}:
                t = prob
                for w in reversed(range(n)):   # fold the register from its last wire
                    t = t.view(psi.shape[0], -1, 2)
                    t = t[..., 0] - t[..., 1] if letters[w] == "Z" else t[..., 0] + t[..., 1]
                E += coef * t.reshape(-1)
            else:
                E += coef * _vdot(psi, _pauli(psi, n, letters)).real
        cols.append(E)
    return torch.stack(cols, 1)


def _seed(psi, n, obs, weights):
    """sum_o w_o H_o psi."""
    lam = torch.zeros_like(psi)
    zsum = None
    for o, w in zip(obs, weights.T):
        for coef, letters in o:
            f = (coef * w)[:, None].to(torch.complex128)
            if set(letters) <= {"I", "Z"}:
                at = [i for i in range(n) if letters[i] == "Z"]
                if zsum is None:
                    zsum = torch.zeros(psi.shape[0], 1 << n, dtype=torch.float64, device=DEV)
                sgn = torch.ones(1, dtype=torch.float64, device=DEV)
                for i in range(at[0] if at else 0, (at[-1] + 1) if at else 0):
                    one = torch.tensor([1.0, -1.0 if letters[i] == "Z" else 1.0], dtype=torch.float64, device=DEV)
                    sgn = (sgn[:, None] * one[None]).reshape(-1)
                lo, hi = (at[0], at[-1] + 1) if at else (0, 0)
                zsum.view(psi.shape[0], 1 << lo, -1, 1 << (n - hi)).add_((coef * w).view(-1, 1, 1, 1) * sgn.view(1, 1, -1, 1))
            else:
                lam.addcmul_(_pauli(psi, n, letters), f.expand_as(psi))
    if zsum is not None:
        lam.addcmul_(psi, zsum.to(torch.complex128))
    return lam


def _angle(g, params, data):
    if g.src == "none":
        return torch.full((1,), g.scale, dtype=torch.float64, device=DEV)
    v = params if g.src == "param" else data
    return g.scale * (v[:, g.idx] if v.dim() == 2 else v[g.idx:g.idx + 1])


def _forward(circuit, params, data, batch, init=None):
    psi = torch.zeros(batch, 1 << circuit.n, dtype=torch.complex128, device=DEV)
    psi[:, 0] = 1
    if init is not None:
        psi = init.to(torch.complex128)
    for g in _simple(circuit.gates):
        psi = _apply(psi, circuit.n, g.wires, _matrix(g, _angle(g, params, data)),
                     _shape(g.op) if g.op != "unitary" else None)
    return psi


def _gradient(circuit, obs, params, data, weights, psi):
    """Gradients of sum w E by the chain of generators, psi the final state (used up)."""
    n, lam = circuit.n, _seed(psi, circuit.n, obs, weights)
    gp = torch.zeros_like(params)
    gd = torch.zeros_like(data) if data is not None else None
    for g in reversed(list(_simple(circuit.gates))):
        if g.src != "none":
            G = _generator(g.op).to(DEV)[None]
            val = _vdot(lam, _apply(psi.clone(), n, g.wires, G, _shape(g.op, True))).imag * g.scale
            to = gp if g.src == "param" else gd
            if to.dim() == 2:
                to[:, g.idx] += val
            else:
                to[g.idx] += val.sum()
        m = _matrix(g, _angle(g, params, data)).mH
        psi = _apply(psi, n, g.wires, m, _shape(g.op))
        lam = _apply(lam, n, g.wires, m, _shape(g.op))
    return gp, gd


def exact(case, seed):
    c, kind = case, case["kind"]
    s = _inputs(c, seed)
    if kind == "measure":
        n, B = c["n"], c["batch"]
        p = torch.view_as_real(s["init"]).double().square().sum(-1)
        shape, at, front = [B], 0, {}
        for w in sorted(s["wires"]):
            shape += [1 << (w - at), 2]
            front[w] = len(shape) - 1
            at = w + 1
        p = p.view(shape + [1 << (n - at)])
        rest = [a for a in range(1, p.dim()) if a not in front.values()]
        p = p.permute([0] + [front[w] for w in s["wires"]] + rest).reshape(B, 1 << len(s["wires"]), -1).sum(-1)
        return [p, None]
    if kind == "qft":
        return [torch.fft.ifft(s["init"].to(torch.complex128), norm="ortho", dim=1)]
    if kind == "multi":
        Es, grads = [], []
        for (circuit, obs), p in zip(_multi_circuits(c), s["params"]):
            psi = _forward(circuit, p, None, 1)
            E = _observe(psi, circuit.n, obs)
            Es.append(E[0])
            grads.append(_gradient(circuit, obs, p, None, torch.ones_like(E), psi)[0])
        return [torch.cat(Es), torch.cat(grads)]
    circuit, obs = _unitary_circuit(c, seed) if kind == "unitary" else _circuit(c)
    params, data, B = s["params"].double(), s["data"].double() if "data" in s else None, c.get("batch", 1)
    if kind == "hessian":
        P, one = circuit.n_params, torch.ones(1, 1, dtype=torch.float64, device=DEV)
        H = torch.zeros(P, P, dtype=torch.float64, device=DEV)
        for q in range(P):
            for sign in (0.5, -0.5):
                t = params.clone()
                t[q] += sign * math.pi
                H[:, q] += sign * _gradient(circuit, obs, t, None, one, _forward(circuit, t, None, 1))[0]
        return [H]
    psi = _forward(circuit, params, data, B)
    E = _observe(psi, circuit.n, obs)
    if kind == "train":
        w = 2 * (E - s["target"]) / E.numel()
        gp, gd = _gradient(circuit, obs, params, data, w, psi)
        return [E, gp] + ([gd] if c["data_grad"] else [])
    if kind == "step":
        return [E, _gradient(circuit, obs, params, None, torch.ones_like(E), psi)[0]]
    return [E, psi]
