"""Fused matrices on the host: phase and permutation gates scale and exchange
rows of the fused matrix instead of being multiplied into it, and gates reach
the planner through one packed record each."""
import itertools

import numpy as np
import pytest

from oracle import sv_oracle as so
from oracle.brute import full_matrix
from paper_2409_14697_amd import binding as B
from svgen import Gate

EPS = 2.0 ** -53


def _product(n, ops):
    u = np.eye(1 << n, dtype=np.complex128)
    for q, m in ops:
        u = full_matrix(m, q, n) @ u
    return u


def _perm_gate(q, perm):
    return Gate("MATRIX", q, matrix=np.eye(1 << len(q))[list(perm)].astype(np.complex128))


@pytest.mark.parametrize("seed", range(6))
def test_phase_and_permutation_products(seed):
    """Products of up to 40 gates, most of them sparse, against the product of
    their definitions: each gate adds at most 16 roundings to an entry of a
    unitary matrix."""
    rng = np.random.default_rng(seed)
    n = 3 + seed % 3
    gates = []
    for i in range(40):
        a, b = (int(x) for x in rng.permutation(n)[:2])
        t = float(rng.uniform(-3, 3))
        gates.append([Gate("CNOT", (a, b)), Gate("CZ", (a, b)), Gate("SWAP", (a, b)), Gate("CPHASE", (a, b), t),
                      Gate("RZZ", (a, b), t), Gate("X", (a,)), Gate("S", (b,)), Gate("RZ", (a,), t), Gate("H", (b,)),
                      _perm_gate((a, b), rng.permutation(4))][int(rng.integers(10))])
    plan = B.Plan(n, "c128", gates, {"mode": "sweep", "max_fuse_qubits": 5})
    got = _product(n, [(q, m) for q, m, _ in plan.export()])
    want = so.circuit_unitary(gates, n)
    assert np.abs(got - want).max() <= 16 * EPS * len(gates)


def test_every_row_permutation():
    """All 24 exchanges of four rows, exactly."""
    base = Gate("MATRIX", (2, 1, 0), matrix=np.arange(64).reshape(8, 8) * (1 + 2j))
    for perm in itertools.permutations(range(4)):
        g = _perm_gate((0, 2), perm)
        plan = B.Plan(3, "c128", [base, g], {"mode": "sweep"})
        (q, m, _), = plan.export()
        assert q == (2, 1, 0)
        want = np.zeros((8, 8), np.complex128)
        for r in range(8):  # row bits (q2 q1 q0); the gate's index is (q0 q2)
            s = perm[((r & 1) << 1) | (r >> 2)]
            want[r] = base.matrix[((s & 1) << 2) | (r & 2) | (s >> 1)]
        assert np.array_equal(m, want)


def test_non_finite_entries_spread_as_in_a_product():
    """A gate with an infinite entry is multiplied in full, and so are the
    others of its circuit (zero times infinity is not a number)."""
    m = np.eye(4, dtype=np.complex128)
    m[0, 0] = np.inf
    plan = B.Plan(3, "c128", [Gate("MATRIX", (0, 1), matrix=m), Gate("CNOT", (1, 0))], {"mode": "sweep"})
    (_, got, _), = plan.export()
    assert np.isnan(got[:, 0]).all()


def test_gate_records():
    """The packed record holds what the fields hold, also where the numbers do
    not fit it."""
    u = np.arange(16).reshape(4, 4) * (1 + 1j)
    gates = [Gate("H", (3,)), Gate("CNOT", (np.int64(2), 1)), Gate("MATRIX", (0, 5), matrix=u),
             Gate("CPHASE", (1, 4), theta=np.float32(1.5))]
    arr, _keep = B.make_gates(gates)
    for sg, g in zip(arr, gates):
        assert sg.kind == B.KIND[g.kind] and sg.nq == len(g.qubits)
        assert list(sg.q) == [int(x) for x in g.qubits] + [-1] * (B.MAXQ - len(g.qubits))
        assert sg.theta == float(g.theta or 0.0)
    assert [arr[2].m[i] for i in range(4)] == [0.0, 0.0, 1.0, 1.0] and not arr[0].m

    class Wide:  # eight qubits, one beyond 32 bits: the count is kept, so the planner refuses it
        kind, qubits, theta, matrix = "MATRIX", tuple(range(7)) + (1 << 40,), 0.0, None

    arr, _keep = B.make_gates([Wide])
    assert arr[0].nq == 8 and list(arr[0].q) == [0, 1, 2, 3, 4, 5]

    class Fractional:
        kind, qubits, theta, matrix = "H", (1.0,), 0.0, None

    with pytest.raises(TypeError):
        B.make_gates([Fractional])
