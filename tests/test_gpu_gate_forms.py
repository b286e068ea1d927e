"""Register-pass gate forms at the places where they can go wrong, against the oracle."""
import numpy as np
import pytest

import workloads as W
from oracle import statevector as O

pytestmark = pytest.mark.gpu
TOL = {"c64": 1e-5, "c128": 1e-12}


def _q():
    import paper_2406_17248_amd as Q
    return Q


def _run(Q, circ, psi, dtype, tile=None):
    s = Q.qsv_state_create(circ["n_qubits"], dtype)
    if tile is not None:
        Q.qsv_state_set_option(s, Q.OPT_TILE_QUBITS, tile)
    Q.qsv_state_set(s, psi)
    Q.qsv_apply_circuit(s, circ)
    return Q.qsv_state_get(s)


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n,tile", [(9, 9), (10, 9), (13, 10), (14, 13)])
def test_controlled_x_moves_every_amplitude(dtype, n, tile):
    """X with up to three controls on slots, lanes, waves and outside qubits: a permutation,
    so the amplitudes come back bit for bit."""
    Q = _q()
    rng = np.random.default_rng(n)
    gates = []
    for _ in range(60):
        qs = rng.permutation(n)
        nc = int(rng.integers(0, 4))
        gates.append(W.gate("X", (qs[0],), ctrls=tuple(qs[1:1 + nc])))
    circ = W.circuit(n, gates)
    psi = W.random_state(n, rng, np.complex64 if dtype == "c64" else np.complex128)
    ref = psi.copy()
    x = np.arange(1 << n)
    for g in gates:
        cm = sum(1 << c for c in g["ctrls"])
        ref = ref[np.where((x & cm) == cm, x ^ (1 << g["targets"][0]), x)]
    assert np.array_equal(_run(Q, circ, psi, dtype, tile), ref)


def _phase_gates(n, count, rng, n_params):
    gates = []
    for _ in range(count):
        kind = str(rng.choice(["RZ", "PS", "RZZ", "Z", "S", "T", "RX"]))
        qs = rng.permutation(n)
        nt = 2 if kind == "RZZ" else 1
        nc = int(rng.integers(0, 3))
        par = ()
        if kind in ("RZ", "PS", "RZZ", "RX"):
            par = ((int(rng.integers(0, n_params)), float(rng.choice([1.0, -0.5])), float(rng.uniform(-1, 1))),)
        gates.append(W.gate(kind, tuple(qs[:nt]), ctrls=tuple(qs[nt:nt + nc]) if kind != "RX" else (), params=par))
    return gates


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n,tile,adj", [(9, 9, 9), (11, 9, 10), (13, 12, 10), (14, 10, 12)])
def test_phase_runs_and_their_gradients(dtype, n, tile, adj):
    """Runs of phases, sign flips and their gradients with targets and controls on slots,
    lanes, waves and outside qubits."""
    Q = _q()
    rng = np.random.default_rng(100 + n)
    circ = W.circuit(n, [W.gate("H", (q,)) for q in range(n)] + _phase_gates(n, 70, rng, 5))
    params = rng.uniform(-np.pi, np.pi, 5)
    ham = W.random_pauli_sum(n, 6, rng)
    s = Q.qsv_state_create(n, dtype)
    Q.qsv_state_set_option(s, Q.OPT_TILE_QUBITS, tile)
    Q.qsv_state_set_option(s, Q.OPT_ADJ_TILE_QUBITS, adj)
    e, g = Q.qsv_expectation_and_grad(s, circ, ham, params)
    e0, g0 = O.grad_adjoint(circ, ham, params)
    scale = max(1.0, sum(abs(c) for c, _ in ham))
    assert abs(e - e0) <= TOL[dtype] * scale
    assert np.max(np.abs(g - g0)) <= TOL[dtype] * scale
    Q.qsv_apply_circuit(s, circ, params)
    assert np.max(np.abs(Q.qsv_state_get(s) - O.simulate(circ, params))) <= TOL[dtype]


def _chain_gates(n, layers, rng):
    """One-qubit gates of every form (identity-like and X-like ones among them) between CZs:
    chains of every pivot, across rounds, passes and normalizations."""
    gates = []
    for layer in range(layers):
        for q in range(n):
            kind = str(rng.choice(["MAT1", "U3", "RX", "RY", "H", "near", "far", "RZ", "S"]))
            if kind in ("near", "far"):
                e = float(rng.choice([0.0, 1e-9, 1e-3]))
                c = np.sqrt(1 - e * e)
                m = np.array([[c, -e], [e, c]]) if kind == "near" else np.array([[e, -c], [c, e]])
                m = np.exp(1j * rng.uniform(0, 6)) * m * np.exp(1j * np.array([0.0, rng.uniform(0, 6)]))
                gates.append(W.gate("MAT1", (q,), matrix=m))
            elif kind == "MAT1":
                gates.append(W.gate(kind, (q,), matrix=W.haar_unitary_2x2(rng)))
            else:
                angles = 3 if kind == "U3" else 1 if kind in ("RX", "RY", "RZ") else 0
                par = tuple((-1, 0.0, float(rng.choice([0.0, np.pi / 2, np.pi, rng.uniform(-7, 7)])))
                            for _ in range(angles))
                gates.append(W.gate(kind, (q,), params=par))
        for a in range(layer % 2, n - 1, 2):
            gates.append(W.gate("Z", (a + 1,), ctrls=(a,)))
        if layer % 7 == 6:  # a chain that a controlled gate ends
            gates.append(W.gate("RY", (0,), ctrls=(n - 1,), params=((-1, 0.0, 0.4),)))
    return gates


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n,tile,layers", [(9, 9, 40), (11, 10, 40), (14, 11, 24), (20, 9, 6), (20, None, 20)])
def test_gate_chains(dtype, n, tile, layers):
    Q = _q()
    rng = np.random.default_rng(n + layers)
    circ = W.circuit(n, _chain_gates(n, layers, rng))
    psi = W.random_state(n, rng, np.complex64 if dtype == "c64" else np.complex128)
    ref = O.simulate(circ, None, psi.astype(np.complex128))
    got = _run(Q, circ, psi, dtype, tile)
    assert np.max(np.abs(got - ref)) <= TOL[dtype]
    assert abs(np.linalg.norm(got.astype(np.complex128)) - np.linalg.norm(psi)) <= 100 * TOL[dtype]


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n", [3, 10])
def test_neighbours_that_share_an_angle(dtype, n):
    """Gates of one kind and of several with equal angles, side by side, and what the reverse
    sweep makes of them: each gets its own numbers."""
    Q = _q()
    gates = [W.gate("H", (q,)) for q in range(n)]
    for kinds in (["RX", "RX", "RY", "RY", "RX"], ["RZ", "PS", "RZ", "RZZ", "RZZ", "RY"], ["PS", "RX", "PS"]):
        for i, k in enumerate(kinds):
            qs = tuple((i + j) % n for j in range(2 if k == "RZZ" else 1))
            gates.append(W.gate(k, qs, params=((0, 1.0, 0.0),)))
        gates.append(W.gate("Z", (1,), ctrls=(0,)))
    circ = W.circuit(n, gates)
    ham = W.random_pauli_sum(n, 5, np.random.default_rng(n))
    s = Q.qsv_state_create(n, dtype)
    e, g = Q.qsv_expectation_and_grad(s, circ, ham, np.array([0.83]))
    e0, g0 = O.grad_adjoint(circ, ham, np.array([0.83]))
    scale = max(1.0, sum(abs(c) for c, _ in ham)) * len(gates)
    assert abs(e - e0) <= TOL[dtype] * scale
    assert np.max(np.abs(g - g0)) <= TOL[dtype] * scale
