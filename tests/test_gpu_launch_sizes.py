"""Batches on both sides of the launch size from which passes leave their tables' warm-up out and
forward passes halve their remaps (1024 tiles): each item does the same arithmetic in the same
order, so its results are the same to the last bit."""
import numpy as np
import pytest

import workloads as W
from oracle import statevector as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def Q():
    import paper_2406_17248_amd as Q
    Q.lib()
    return Q


# tiles of 10 (reverse) and 12 (forward) qubits in complex64, of 11 in complex128
@pytest.mark.parametrize("dtype,n,edge", [("c64", 11, 512), ("c64", 13, 128), ("c64", 13, 512), ("c128", 12, 512)])
@pytest.mark.parametrize("phases", [False, True])
def test_items_do_not_depend_on_the_launch(Q, dtype, n, edge, phases):
    rng = np.random.default_rng(n + edge)
    gates = [W.gate("H", (q,)) for q in range(n)]
    for layer in range(2):
        gates += [W.gate("RZZ", (q, (q + 3) % n), params=((layer, 2.0, 0.0),)) for q in range(n)]
        if phases:
            gates += [W.gate("RZ", (q,), params=((4 + q, 1.0, 0.0),)) for q in range(n)]
        gates += [W.gate("RX", (q,), params=((2 + layer, 1.0, 0.0),)) for q in range(n)]
    circ = W.circuit(n, gates)
    ham = [(0.5, ((q, "Z"), ((q + 1) % n, "Z"))) for q in range(n)] + [(0.3, ((q, "X"),)) for q in range(0, n, 4)]
    params = rng.uniform(-np.pi, np.pi, (edge + 1, 4 + n if phases else 4))
    s = Q.qsv_state_create(n, dtype)
    small = Q.qsv_expectation_and_grad_batch(s, circ, ham, params[:edge])
    large = Q.qsv_expectation_and_grad_batch(s, circ, ham, params)
    assert np.array_equal(small[0], large[0][:edge])
    assert np.array_equal(small[1], large[1][:edge])
    e0, g0 = O.grad_adjoint(circ, ham, params[edge])
    tol = (1e-5 if dtype == "c64" else 1e-12) * sum(abs(c) for c, _ in ham)
    assert abs(large[0][edge] - e0) <= tol
    assert np.max(np.abs(large[1][edge] - g0)) <= tol * n
