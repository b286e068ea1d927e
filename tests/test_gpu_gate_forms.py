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
