"""Pauli sums at their limits on the GPU: coefficients near the end of the range."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def Q():
    import paper_2406_17248_amd as Q
    Q.lib()
    return Q


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n", [8, 12, 19])
def test_largest_coefficients(Q, dtype, n):
    """Two x masks in one pass; twice the larger coefficient is not a finite number.  <X> =
    sin(0.6) and <Y> = 0 on every qubit."""
    c = 1.7e308
    h = [(1.0, ((0, "X"),)), (c, ((n - 1, "X"),)), (-0.1 * c, ((n - 1, "Y"),))]
    circ = W.circuit(n, [W.gate("RY", (q,), params=((-1, 0.0, 0.6),)) for q in range(n)])
    s = Q.qsv_state_create(n, dtype)
    Q.qsv_apply_circuit(s, circ)
    e = Q.qsv_expectation(s, h).real
    assert np.isfinite(e)
    # n gates round every amplitude, twice in the sum
    assert abs(e / c - np.sin(0.6)) <= 2 * n * np.finfo(np.float32 if dtype == "c64" else np.float64).eps
    assert Q.qsv_expectation_noalloc(s, h).real == e
