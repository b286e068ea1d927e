"""Pauli sums of several x masks on states of 22 to 24 qubits, tiled and gathered, against plain
torch in complex128, with bounds in which one term of the sum shows."""
import math

import numpy as np
import pytest
import torch  # before the library: one HIP runtime for both

import workloads as W

pytestmark = pytest.mark.gpu
EPS = {"c64": 2.0 ** -24, "c128": 2.0 ** -53}


@pytest.fixture(scope="module")
def Q():
    import paper_2406_17248_amd as Q
    Q.lib()
    return Q


def pauli_times(a, n, factors):
    """A Pauli string times the complex128 state `a`, by flips and halves of its 2 x .. x 2 view."""
    t = a.view([2] * n)
    flips = [n - 1 - q for q, p in factors if p in "XY"]
    out = torch.flip(t, flips) if flips else t.clone()
    for q, p in factors:
        if p != "X":
            out.select(n - 1 - q, 1).neg_()
        if p == "Y":
            out.mul_(-1j)
    return out.reshape(-1)


def product_state(n, rng, device):
    """Every qubit at its own place on the Bloch sphere, all three components of 0.3 to 0.8: a string of
    k factors has an expectation of 0.3^k at least.  (state, components)"""
    a = torch.ones(1, dtype=torch.complex128, device=device)
    bloch = []
    for _ in range(n):
        v = 0.5 + 0.3 * rng.uniform(0.0, 1.0, 3)
        v /= np.linalg.norm(v)
        bloch.append(dict(zip("XYZ", v)))
        th, ph = math.acos(v[2]), math.atan2(v[1], v[0])
        one = torch.tensor([math.cos(th / 2), math.sin(th / 2) * complex(math.cos(ph), math.sin(ph))],
                           dtype=torch.complex128, device=device)
        a = torch.outer(one, a).reshape(-1)  # qubit 0 is the lowest bit
    return a, bloch


def the_sum(n, rng):
    h = W.random_pauli_sum(n, 24, rng, max_locality=4)
    h += [(0.4, ((q, p), (q + 1, p))) for q in range(n - 1) for p in "XYZ"]
    h += [(0.7, ((0, "X"),)), (-0.3, ((0, "X"), (n - 1, "Y"))), (0.2, ((0, "X"), (n - 1, "X"))), (0.3, ((n - 2, "Z"),))]
    return [h[i] for i in rng.permutation(len(h))]


# tiles from 24 qubits (complex64) and 23 (complex128) on, gathers below
@pytest.mark.parametrize("dtype,n", [("c64", 23), ("c64", 24), ("c128", 22), ("c128", 23)])
def test_sums_of_many_masks(Q, dtype, n):
    from paper_2406_17248_amd import torch_layer as TL
    rng = np.random.default_rng(50 + n)
    h = the_sum(n, rng)
    scale = sum(abs(c) for c, _ in h)
    prod, bloch = product_state(n, rng, "cuda")
    a = prod.to(torch.complex64 if dtype == "c64" else torch.complex128)
    b = torch.empty_like(a)
    s, d = TL.state_from_tensor(a), TL.state_from_tensor(b)
    Q.qsv_apply_pauli_sum(d, s, h)
    e = Q.qsv_expectation(s, h)
    wide = a.to(torch.complex128)
    ref = torch.zeros_like(wide)
    for c, factors in h:
        ref.add_(pauli_times(wide, n, factors), alpha=c)
    # every launch (a dozen) rounds H psi once, the reference every term once
    bound = (16 * EPS[dtype] + (len(h) + 4) * EPS["c128"]) * scale * float(wide.abs().max())
    err = float((b.to(torch.complex128) - ref).abs().max())
    assert err <= bound
    # energies are summed in double in both types: of exact products, one rounding per level of the sums
    e_ref = float(torch.vdot(wide, ref).real)
    assert abs(e.real - e_ref) <= 200 * EPS["c128"] * scale
    # ... and are the product state's (to the rounding of its amplitudes)
    e_bloch = sum(c * math.prod(bloch[q][p] for q, p in f) for c, f in h)
    assert abs(e.real - e_bloch) <= (4 * EPS[dtype] + 4 * n * EPS["c128"]) * scale
    # both bounds see one of the neighbour terms: its smallest change of the largest amplitudes and
    # of the energy
    assert bound < 0.1 * 0.4 * float(wide.abs().max()) and 4 * EPS[dtype] * scale < 0.1 * 0.4 * 0.3 ** 2


@pytest.mark.parametrize("n", [23, 24, 25])
def test_gradients_of_sums_of_many_masks_c64(Q, n):
    """Complex64 gradients keep the groups in order, in gathers, also where states are large."""
    rng = np.random.default_rng(n)
    h = the_sum(n, rng)
    scale = sum(abs(c) for c, _ in h)
    gates = [W.gate("RY", (q,), params=((0, 1.0, 0.1 * q),)) for q in range(n)]
    gates += [W.gate("Z", (q + 1,), ctrls=(q,)) for q in range(0, n - 1, 2)]
    gates += [W.gate("RX", (q,), params=((1, 1.0, 0.2 * q),)) for q in range(0, n, 5)]
    params = np.array([0.4, 0.9])
    s = Q.qsv_state_create(n, "c64")
    e, g = Q.qsv_expectation_and_grad(s, W.circuit(n, gates), h, params)

    def turn(v, q, p, angle):  # exp(-i angle P / 2) v
        return math.cos(angle / 2) * v - 1j * math.sin(angle / 2) * pauli_times(v, n, ((q, p),))

    def step(v, gate, sign):
        q = gate["targets"][0]
        if gate["ctrls"]:
            w = v.view([2] * n)
            w.select(n - 1 - gate["ctrls"][0], 1).select(n - 1 - q - (q < gate["ctrls"][0]), 1).neg_()
            return v
        i, f, c = gate["params"][0]
        return turn(v, q, gate["kind"][1], sign * (c + f * params[i]))

    psi = torch.zeros(1 << n, dtype=torch.complex128, device="cuda")
    psi[0] = 1
    for gate in gates:
        psi = step(psi, gate, 1)
    lam = torch.zeros_like(psi)
    for c, factors in h:
        lam.add_(pauli_times(psi, n, factors), alpha=c)
    e_ref = float(torch.vdot(psi, lam).real)
    g_ref = np.zeros(2)
    for gate in reversed(gates):
        if not gate["ctrls"]:
            g_ref[gate["params"][0][0]] += float(torch.vdot(lam, pauli_times(psi, n, ((gate["targets"][0], gate["kind"][1]),))).imag)
        psi, lam = step(psi, gate, -1), step(lam, gate, -1)
    # amplitudes are rounded by every gate on both sides and by every group: in the mean, not all one way
    tol = EPS["c64"] * scale * math.sqrt(len(gates) + len(h))
    assert abs(e - e_ref) <= 4 * tol
    assert np.max(np.abs(g - g_ref)) <= 4 * tol * math.sqrt(n)
