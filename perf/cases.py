"""The work that programs have this engine do, as timed cases.

Each case is one call sequence through the public entry points:

* ``apply``     a circuit applied to a state (from |0...0>, or from a given state), with the
                expectation of sum_i Z_i where ``sum_z`` asks for it
* ``expect``    <psi|H|psi> of a Pauli sum on a given state
* ``hpsi``      H|psi> of a Pauli sum
* ``grad``      energies and adjoint gradients of a batch of parameter sets of one circuit
* ``train``     forward and backward of the trainable torch layer
* ``uneven``    energies and gradients of many circuits of different sizes in one call

``listed()`` holds the sizes that stand for each use, ``draw()`` more of the same ranges.
"""

from __future__ import annotations

import math

import numpy as np
import torch

import paper_2406_17248_amd as Q
from paper_2406_17248_amd import torch_layer as TL

KINDS = ("X", "Y", "Z", "H", "S", "SDG", "T", "TDG", "RX", "RY", "RZ", "PS", "RXX", "RYY", "RZZ", "U3",
         "SWAP", "MAT1", "MAT2")
TWO_TARGETS = ("RXX", "RYY", "RZZ", "SWAP", "MAT2")
ONE_ANGLE = ("RX", "RY", "RZ", "PS", "RXX", "RYY", "RZZ")


def listed():
    return [
        # A few gates of every kind on a handful of qubits: a test or a notebook cell; latency only.
        dict(name="apply_mixed_n6_c128", do="apply", circuit="mixed", n=6, gates=40, dtype="c128"),
        # The 10-qubit hardware-efficient ansatz with a ZZ chain: one optimizer step's energy and gradient.
        dict(name="grad_hea_n10_c128", do="grad", circuit="hea", n=10, depth=4, batch=1, ham="zz_chain", dtype="c128"),
        # A 50-term Hamiltonian of 1- to 4-local strings on a small state.
        dict(name="expect_random_n11_c128", do="expect", n=11, ham="random", terms=50, dtype="c128"),
        # One training step of the torch layer: forward and backward of a 14-qubit ansatz.
        dict(name="train_hea_n14_c64", do="train", circuit="hea", n=14, depth=3, ham="random", terms=24, dtype="c64"),
        # QAOA angles of many starting points at once on a 16-qubit graph (an odd batch).
        dict(name="grad_qaoa_n16_b33_c64", do="grad", circuit="qaoa", n=16, depth=6, batch=33, ham="maxcut",
             dtype="c64"),
        # Circuits of 8 to 20 qubits, each with its own 50-term Hamiltonian, in one graph launch.
        dict(name="uneven_48_c64", do="uneven", count=48, n_min=8, n_max=20, depth_min=2, depth_max=10, terms=50,
             dtype="c64"),
        # Every gate kind, with controls, on a 23-qubit given state.
        dict(name="apply_mixed_n23_c64", do="apply", circuit="mixed", n=23, gates=120, dtype="c64"),
        # H|psi> of a 50-term Hamiltonian (Krylov and imaginary-time steps, variances).
        dict(name="hpsi_random_n24_c64", do="hpsi", n=24, ham="random", terms=50, dtype="c64"),
        # QAOA p = 8 on the 24-node graph: energies and gradients of 8 parameter sets.
        dict(name="grad_qaoa_n24_b8_c128", do="grad", circuit="qaoa", n=24, depth=8, batch=8, ham="maxcut",
             dtype="c128"),
        # Energy of a Heisenberg chain with a field on a 26-qubit state.
        dict(name="expect_heisenberg_n26_c128", do="expect", n=26, ham="heisenberg", terms=0, dtype="c128"),
        # Random brick circuit, odd size, single precision.
        dict(name="apply_brick_n27_c64", do="apply", circuit="brick", n=27, depth=20, dtype="c64", sum_z=True),
        # The benchmark step: 30 qubits, depth 20, double precision, then <sum Z>.
        dict(name="apply_brick_n30_c128", do="apply", circuit="brick", n=30, depth=20, dtype="c128", sum_z=True),
    ]


def draw(rng):
    do = rng.choice(["apply", "apply", "apply", "grad", "grad", "grad", "expect", "hpsi", "train", "uneven"])
    dtype = rng.choice(["c64", "c128"])
    if do == "apply":
        kind = rng.choice(["mixed", "brick", "brick", "hea"])
        if kind == "mixed":
            return dict(do=do, circuit=kind, n=rng.randint(2, 25), gates=int(round(10 ** rng.uniform(1.0, 2.3))),
                        dtype=dtype)
        return dict(do=do, circuit=kind, n=rng.randint(4, 28), depth=rng.randint(1, 20), dtype=dtype,
                    sum_z=rng.random() < 0.5)
    if do in ("expect", "hpsi"):
        ham = rng.choice(["random", "random", "heisenberg", "ising", "sum_z"])
        return dict(do=do, n=rng.randint(3, 26 if do == "expect" else 25), ham=ham,
                    terms=int(round(10 ** rng.uniform(0.0, 2.0))), dtype=dtype)
    if do == "grad":
        if rng.random() < 0.5:
            n = rng.randint(3, 20)
            return dict(do=do, circuit="hea", n=n, depth=rng.randint(1, 6), batch=rng.randint(1, max(1, 24 - n)),
                        ham=rng.choice(["zz_chain", "random", "heisenberg"]), terms=rng.randint(5, 50), dtype=dtype)
        n = rng.randint(5, 23)
        most = min(64.0, 2.0 ** (26 - n))
        return dict(do=do, circuit="qaoa", n=n, depth=rng.randint(1, 8),
                    batch=int(round(math.exp(rng.uniform(0.0, math.log(most))))), ham="maxcut", dtype=dtype)
    if do == "train":
        return dict(do=do, circuit="hea", n=rng.randint(4, 18), depth=rng.randint(1, 5),
                    ham=rng.choice(["zz_chain", "random", "heisenberg"]), terms=rng.randint(4, 50), dtype=dtype)
    lo = rng.randint(4, 12)
    return dict(do=do, count=rng.randint(3, 64), n_min=lo, n_max=rng.randint(lo, 20), depth_min=1,
                depth_max=rng.randint(2, 10), terms=rng.randint(1, 50), dtype=dtype)


# ---------------------------------------------------------------------------------------------
# Circuits and Hamiltonians as the plain descriptions that the package takes
# ---------------------------------------------------------------------------------------------
def _gate(kind, targets, ctrls=(), params=(), matrix=None):
    return {"kind": kind, "targets": tuple(targets), "ctrls": tuple(ctrls), "params": tuple(params), "matrix": matrix}


def _haar(d, rng):
    z = rng.standard_normal((d, d)) + 1j * rng.standard_normal((d, d))
    q, r = np.linalg.qr(z)
    return q * (np.diagonal(r) / np.abs(np.diagonal(r)))


def _brick(n, depth, rng):
    gs = []
    for layer in range(depth):
        gs += [_gate("MAT1", (q,), matrix=_haar(2, rng)) for q in range(n)]
        gs += [_gate("Z", (a + 1,), (a,)) for a in range(layer % 2, n - 1, 2)]
    return gs


def _hea(n, depth):
    gs = []
    for k in range(depth):
        for q in range(n):
            gs.append(_gate("RY", (q,), params=((2 * n * k + q, 1.0, 0.0),)))
            gs.append(_gate("RZ", (q,), params=((2 * n * k + n + q, 1.0, 0.0),)))
        gs += [_gate("X", (q + 1,), (q,)) for q in range(n - 1)]
    return gs


def _graph(n, rng):
    """A random 3-regular graph (4-regular for an odd number of nodes) by pairing."""
    d = min(3 if n % 2 == 0 else 4, n - 1)
    while True:
        ends = rng.permutation(np.repeat(np.arange(n), d)).reshape(-1, 2)
        edges = {(int(min(a, b)), int(max(a, b))) for a, b in ends}
        if len(edges) == n * d // 2 and all(a != b for a, b in edges):
            return sorted(edges)


def _qaoa(n, depth, edges):
    gs = [_gate("H", (q,)) for q in range(n)]
    for k in range(depth):
        gs += [_gate("RZZ", e, params=((k, 2.0, 0.0),)) for e in edges]
        gs += [_gate("RX", (q,), params=((depth + k, 1.0, 0.0),)) for q in range(n)]
    return gs


def _mixed(n, count, rng):
    gs = []
    for i in range(count):
        kind = KINDS[int(rng.integers(len(KINDS)))]
        qs = [int(q) for q in rng.permutation(n)]
        nt = 2 if kind in TWO_TARGETS else 1
        nc = min(int(rng.integers(0, 3)), n - nt) if rng.random() < 0.4 else 0
        angles = 3 if kind == "U3" else 1 if kind in ONE_ANGLE else 0
        params = [(-1, 0.0, float(rng.uniform(-math.pi, math.pi))) for _ in range(angles)]
        mat = _haar(2 if kind == "MAT1" else 4, rng) if kind in ("MAT1", "MAT2") else None
        gs.append(_gate(kind, qs[:nt], qs[nt:nt + nc], params, mat))
    return gs


def _random_terms(n, count, rng):
    terms = []
    for _ in range(count):
        k = int(rng.integers(1, min(4, n) + 1))
        qs = rng.permutation(n)[:k]
        terms.append((float(rng.standard_normal()), tuple((int(q), "XYZ"[int(rng.integers(3))]) for q in qs)))
    return terms


def _hamiltonian(case, rng, edges=None):
    n, kind = case["n"], case["ham"]
    if kind == "random":
        return _random_terms(n, case["terms"], rng)
    if kind == "sum_z":
        return [(1.0, ((q, "Z"),)) for q in range(n)]
    if kind == "zz_chain":
        return [(1.0, ((q, "Z"), (q + 1, "Z"))) for q in range(n - 1)]
    if kind == "ising":  # transverse field
        j, g = rng.uniform(0.5, 1.5, 2)
        return [(-j, ((q, "Z"), (q + 1, "Z"))) for q in range(n - 1)] + [(-g, ((q, "X"),)) for q in range(n)]
    if kind == "heisenberg":
        jx, jy, jz, hz = rng.uniform(0.5, 1.5, 4)
        terms = []
        for q in range(n - 1):
            terms += [(c, ((q, p), (q + 1, p))) for c, p in ((jx, "X"), (jy, "Y"), (jz, "Z"))]
        return terms + [(hz, ((q, "Z"),)) for q in range(n)]
    return [(0.5 * len(edges), ())] + [(-0.5, ((a, "Z"), (b, "Z"))) for a, b in edges]  # maxcut


def _shapes(case):
    """Qubits and depth of each circuit of an uneven batch: of the case, whatever the seed."""
    rng = np.random.default_rng([case["count"], case["n_min"], case["n_max"], case["depth_max"]])
    return [(int(rng.integers(case["n_min"], case["n_max"] + 1)),
             int(rng.integers(case["depth_min"], case["depth_max"] + 1))) for _ in range(case["count"])]


def _n_params(gates):
    return max([i + 1 for g in gates for i, _, _ in g["params"]], default=0)


def _describe(case, seed):
    """The inputs of a case as plain descriptions: circuit(s), Hamiltonian(s), parameters."""
    rng = np.random.default_rng(seed)
    d = {}
    if case["do"] == "uneven":
        d["circuits"], d["hams"], params = [], [], []
        for n, depth in _shapes(case):
            gates = _hea(n, depth)
            d["circuits"].append({"n_qubits": n, "gates": gates})
            d["hams"].append(_random_terms(n, case["terms"], rng))
            params.append(rng.uniform(0.0, 2 * math.pi, _n_params(gates)))
        d["params"] = np.concatenate(params)
        return d
    edges = None
    if "circuit" in case:
        if case["circuit"] == "brick":
            gates = _brick(case["n"], case["depth"], rng)
        elif case["circuit"] == "hea":
            gates = _hea(case["n"], case["depth"])
        elif case["circuit"] == "mixed":
            gates = _mixed(case["n"], case["gates"], rng)
        else:
            edges = _graph(case["n"], rng)
            gates = _qaoa(case["n"], case["depth"], edges)
        d["circuit"] = {"n_qubits": case["n"], "gates": gates}
        top = math.pi if case["circuit"] == "qaoa" else 2 * math.pi
        d["params"] = rng.uniform(0.0, top, (case.get("batch", 1), _n_params(gates)))
    if "ham" in case or case.get("sum_z"):
        d["ham"] = _hamiltonian(case if "ham" in case else dict(case, ham="sum_z"), rng, edges)
    return d


def _random_state(n, dtype, seed, device):
    g = torch.Generator(device=device).manual_seed(seed)
    real = torch.float32 if dtype == "c64" else torch.float64
    v = torch.view_as_complex(torch.randn(1 << n, 2, generator=g, dtype=real, device=device))
    return v / math.sqrt(2.0 ** (n + 1))


def _buffer(n, dtype):
    return torch.zeros(1 << n, dtype=torch.complex64 if dtype == "c64" else torch.complex128, device="cuda")


def _given_state(case):
    return case["do"] in ("expect", "hpsi") or case.get("circuit") == "mixed"


# ---------------------------------------------------------------------------------------------
def prepare(case, seed):
    d = _describe(case, seed)
    s = {"case": case}
    if case["do"] == "uneven":
        s["batch"] = Q.qsv_batch_create(d["circuits"], d["hams"], case["dtype"])
        s["params"] = d["params"]
        return s
    if case["do"] == "train":
        s["layer"] = TL.AnsatzExpectation(d["circuit"], d["ham"], dtype=case["dtype"], init=d["params"][0])
        return s
    if "circuit" in d:
        s["circuit"], s["params"] = Q.Circuit(d["circuit"]), d["params"]
    if "ham" in d:
        s["ham"] = Q.PauliSum(d["ham"])
    if _given_state(case):
        s["input"] = TL.state_from_tensor(_random_state(case["n"], case["dtype"], seed, "cuda"))
    if case["do"] in ("apply", "hpsi"):
        s["amps"] = _buffer(case["n"], case["dtype"])
        s["state"] = TL.state_from_tensor(s["amps"])
    elif case["do"] == "grad":
        s["state"] = Q.qsv_state_create(case["n"], case["dtype"])
    return s


def run(state):
    case = state["case"]
    if case["do"] == "apply":
        if "input" in state:
            Q.qsv_state_copy(state["state"], state["input"])
        else:
            Q.qsv_state_reset(state["state"])
        Q.qsv_apply_circuit(state["state"], state["circuit"], state["params"][0])
        out = {"psi": state["amps"]}
        if "ham" in state:
            out["E"] = Q.qsv_expectation(state["state"], state["ham"]).real
        return out
    if case["do"] == "expect":
        e = Q.qsv_expectation(state["input"], state["ham"])
        return {"E": e.real}
    if case["do"] == "hpsi":
        Q.qsv_apply_pauli_sum(state["state"], state["input"], state["ham"])
        return {"hpsi": state["amps"]}
    if case["do"] == "grad":
        e, g = Q.qsv_expectation_and_grad_batch(state["state"], state["circuit"], state["ham"], state["params"])
        return {"E": e, "grad": g}
    if case["do"] == "train":
        layer = state["layer"]
        layer.weight.grad = None
        e = layer()
        e.backward()
        return {"E": e.detach(), "grad": layer.weight.grad}
    e, g = Q.qsv_batch_expectation_and_grad(state["batch"], state["params"])
    return {"E": e, "grad": g}


# ---------------------------------------------------------------------------------------------
# Work: bytes and flop that one pass cannot do without.  The state is read and written once
# however many gates run on it; a one-qubit matrix costs 14 flop per amplitude, a two-qubit one
# 30, a phase 6; undoing it on psi and lambda twice that, a gradient term 4 per amplitude.
# ---------------------------------------------------------------------------------------------
def _gate_flops(kind):
    if kind in ("X", "Z", "SWAP"):  # sign flips and moves
        return 0
    if kind in ("RXX", "RYY", "MAT2"):
        return 30
    if kind in ("S", "SDG", "T", "TDG", "RZ", "PS", "RZZ"):
        return 6
    return 14


def _circuit_flops(circuit, n, depth, gates=0):
    """(flop per amplitude of the gates, number of parameterized gates)"""
    if circuit == "brick":
        return 14 * n * depth, 0
    if circuit == "hea":
        return (14 + 6) * n * depth, 2 * n * depth
    if circuit == "qaoa":  # the equal phases of a cost layer are one
        d = min(3 if n % 2 == 0 else 4, n - 1)
        return 14 * n + depth * (6 + 14 * n), depth * (n * d // 2 + n)
    return gates * sum(_gate_flops(k) for k in KINDS) / len(KINDS), 0


def _ham_flops(ham, n, terms):
    """flop per amplitude: |amplitude|^2 and one product and sum for each term's share"""
    if ham == "random":
        return 3 + 4 * terms
    return 3 + 2 * {"sum_z": n, "zz_chain": n - 1, "maxcut": 2 * n, "ising": 2 * n - 1, "heisenberg": 4 * n - 3}[ham]


def work(case):
    size = 8 if case["dtype"] == "c64" else 16
    if case["do"] == "uneven":
        parts = [dict(do="grad", circuit="hea", n=n, depth=d, batch=1, ham="random", terms=case["terms"],
                      dtype=case["dtype"]) for n, d in _shapes(case)]
        works = [work(p) for p in parts]
        return {"bytes": sum(w["bytes"] for w in works), "flops": sum(w["flops"] for w in works)}
    amps = 2.0 ** case["n"] * case.get("batch", 1)
    flops, params = 0.0, 0
    if "circuit" in case:
        flops, params = _circuit_flops(case["circuit"], case["n"], case.get("depth", 0), case.get("gates", 0))
    if case["do"] in ("grad", "train"):
        # one value of the state at a time: psi written by the forward circuit, psi and lambda by the reverse one
        flops = 3 * flops + 4 * params + _ham_flops(case["ham"], case["n"], case.get("terms", 0))
        return {"bytes": 3 * amps * size, "flops": flops * amps}
    if case["do"] == "apply":
        sides = 2 if _given_state(case) else 1
        if case.get("sum_z"):
            flops += _ham_flops("sum_z", case["n"], 0)
        return {"bytes": sides * amps * size, "flops": flops * amps}
    flops = _ham_flops(case["ham"], case["n"], case["terms"])
    return {"bytes": (2 if case["do"] == "hpsi" else 1) * amps * size, "flops": flops * amps}


# ---------------------------------------------------------------------------------------------
# The same in complex128 by plain torch
# ---------------------------------------------------------------------------------------------
def _matrix(g, params):
    """The gate's 2x2 / 4x4 matrix (row/column bit b of a 4x4 is targets[b])."""
    k = g["kind"]
    a = [c + f * params[i] if i >= 0 else c for i, f, c in g["params"]]
    pauli = {"X": np.array([[0, 1], [1, 0]]), "Y": np.array([[0, -1j], [1j, 0]]), "Z": np.diag([1.0, -1.0])}
    if k in pauli:
        return pauli[k].astype(complex)
    if k == "H":
        return np.array([[1, 1], [1, -1]], dtype=complex) / math.sqrt(2.0)
    if k in ("S", "SDG", "T", "TDG", "PS"):
        angle = {"S": math.pi / 2, "SDG": -math.pi / 2, "T": math.pi / 4, "TDG": -math.pi / 4}.get(k)
        return np.diag([1.0, np.exp(1j * (a[0] if angle is None else angle))])
    if k in ("RX", "RY", "RZ"):
        return math.cos(a[0] / 2) * np.eye(2) - 1j * math.sin(a[0] / 2) * pauli[k[1]]
    if k in ("RXX", "RYY", "RZZ"):
        return math.cos(a[0] / 2) * np.eye(4) - 1j * math.sin(a[0] / 2) * np.kron(pauli[k[1]], pauli[k[1]])
    if k == "U3":
        rz = [np.diag([np.exp(-0.5j * t), np.exp(0.5j * t)]) for t in (a[1], a[2])]
        c, s = math.cos(a[0] / 2), math.sin(a[0] / 2)
        return rz[0] @ np.array([[c, -s], [s, c]]) @ rz[1]
    if k == "SWAP":
        return np.eye(4, dtype=complex)[[0, 2, 1, 3]]
    return np.asarray(g["matrix"], dtype=complex)


def _apply(psi, n, g, m):
    """psi <- (controlled) m psi on g's targets, in place."""
    t = psi.view([2] * n)
    at = [slice(None)] * n
    for c in g["ctrls"]:
        at[n - 1 - c] = 1
    views = []
    for b in range(len(m)):
        w = list(at)
        for j, q in enumerate(g["targets"]):
            w[n - 1 - q] = (b >> j) & 1
        views.append(t[tuple(w)])
    if np.count_nonzero(m - np.diag(np.diagonal(m))) == 0:
        for b, v in enumerate(views):
            if m[b, b] != 1:
                v.mul_(complex(m[b, b]))
        return
    old = [v.clone() for v in views]
    for b, v in enumerate(views):
        v.copy_(sum(complex(m[b, c]) * old[c] for c in range(len(m)) if m[b, c] != 0))


def _pauli(psi, n, factors):
    """The Pauli string applied to psi."""
    t = psi.view([2] * n)
    flips = [n - 1 - q for q, p in factors if p in "XY"]
    out = t.flip(flips) if flips else t.clone()
    for q, p in factors:
        if p == "X":
            continue
        half = out.select(n - 1 - q, 1)
        half.neg_()
        if p == "Y":  # rows of Y: -i on the 0 half, i on the 1 half
            out.mul_(-1j)
    return out.reshape(-1)


def _apply_sum(psi, n, terms):
    out = torch.zeros_like(psi)
    diag = torch.zeros(psi.numel(), dtype=torch.float64, device=psi.device)
    x = torch.arange(psi.numel(), device=psi.device)
    for c, factors in terms:
        if all(p == "Z" for _, p in factors):
            sign = torch.ones_like(diag)
            for q, _ in factors:
                sign *= (1 - 2 * (x >> q & 1))
            diag += c * sign
        else:
            out += c * _pauli(psi, n, factors)
    return out.addcmul_(psi, diag.to(psi.dtype))


def _layers(gates):
    """The gates, with each run of equally bound RZZ as one entry ("cost", run)."""
    out = []
    for g in gates:
        if g["kind"] == "RZZ" and out and out[-1][0] == "cost" and out[-1][1][0]["params"] == g["params"]:
            out[-1][1].append(g)
        else:
            out.append(("cost", [g]) if g["kind"] == "RZZ" else ("gate", g))
    return out


def _energy_and_grad(circuit, terms, params, device):
    """E and dE/dparams: forward, lambda = H psi, then the gates undone one by one on both."""
    n, p = circuit["n_qubits"], [float(v) for v in params]
    psi = torch.zeros(1 << n, dtype=torch.complex128, device=device)
    psi[0] = 1
    x = torch.arange(1 << n, device=device)
    layers, sums = _layers(circuit["gates"]), {}

    def zz(run):  # sum of the run's Z Z eigenvalues
        key = tuple(g["targets"] for g in run)
        if key not in sums:
            sums[key] = sum(1 - 2 * ((x >> a ^ x >> b) & 1) for a, b in key).to(torch.float64)
        return sums[key]

    def angle(g):
        i, f, c = g["params"][0]
        return c + (f * p[i] if i >= 0 else 0.0)

    for kind, g in layers:
        if kind == "cost":
            psi.mul_(torch.exp(-0.5j * angle(g[0]) * zz(g)))
        else:
            _apply(psi, n, g, _matrix(g, p))
    lam = _apply_sum(psi, n, terms)
    energy = float(torch.vdot(psi, lam).real)
    grad = np.zeros(len(p))
    for kind, g in reversed(layers):
        first = g[0] if kind == "cost" else g
        if first["params"] and first["params"][0][0] >= 0:
            i, f, _ = first["params"][0]
            gen = zz(g) * psi if kind == "cost" else _pauli(psi, n, tuple((q, g["kind"][1]) for q in g["targets"]))
            grad[i] += f * float(torch.vdot(lam, gen).imag)
        for v in (psi, lam):
            if kind == "cost":
                v.mul_(torch.exp(0.5j * angle(g[0]) * zz(g)))
            else:
                _apply(v, n, g, _matrix(g, p).conj().T)
    return energy, grad


def exact(case, seed):
    device = "cuda" if torch.cuda.is_available() else "cpu"
    if case.get("n", 0) > 27:
        return None
    d = _describe(case, seed)
    if case["do"] in ("grad", "train"):
        got = [_energy_and_grad(d["circuit"], d["ham"], p, device) for p in d["params"]]
        e, g = np.array([v[0] for v in got]), np.array([v[1] for v in got])
        if case["do"] == "train":
            return {"E": torch.tensor(e[0]), "grad": torch.tensor(g[0])}
        return {"E": e, "grad": g}
    if case["do"] == "uneven":
        es, gs, at = [], [], 0
        for c, h in zip(d["circuits"], d["hams"]):
            k = _n_params(c["gates"])
            e, g = _energy_and_grad(c, h, d["params"][at:at + k], device)
            es.append(e)
            gs.append(g)
            at += k
        return {"E": np.array(es), "grad": np.concatenate(gs)}
    n = case["n"]
    if _given_state(case):
        psi = _random_state(n, case["dtype"], seed, device).to(torch.complex128)
    else:
        psi = torch.zeros(1 << n, dtype=torch.complex128, device=device)
        psi[0] = 1
    if case["do"] == "expect":
        return {"E": float(torch.vdot(psi, _apply_sum(psi, n, d["ham"])).real)}
    if case["do"] == "hpsi":
        return {"hpsi": _apply_sum(psi, n, d["ham"])}
    for g in d["circuit"]["gates"]:
        _apply(psi, n, g, _matrix(g, d["params"][0]))
    out = {"psi": psi}
    if "ham" in d:
        out["E"] = float(torch.vdot(psi, _apply_sum(psi, n, d["ham"])).real)
    return out
