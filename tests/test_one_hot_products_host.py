"""Fused products with matrices whose rows hold a single one each, whether the
rows differ (a permutation) or repeat (projectors, resets): the library does
not check unitarity, so both are planned as the products they are."""
import itertools
import multiprocessing as mp

import numpy as np
import pytest

from oracle import sv_oracle as so
from oracle.brute import full_matrix
from paper_2409_14697_amd import binding as B
from svgen import Gate

EPS = 2.0 ** -53
TIME_LIMIT = 60.0


def _rows(q, src):
    return Gate("MATRIX", tuple(q), matrix=np.eye(len(src))[list(src)].astype(np.complex128))


def _circuits():
    """(n, gates): after dense one- and two-qubit gates every row map of one
    qubit and every row map of two, fused into ops of one to five qubits."""
    for src in itertools.product(range(2), repeat=2):
        yield 7, [Gate("H", (0,)), _rows((0,), src)]
        yield 7, [Gate("RY", (1,), 0.7), Gate("CNOT", (1, 5)), _rows((5,), src), Gate("RX", (5,), 0.3)]
        yield 7, [Gate("RY", (q,), 0.2 + q) for q in range(7)] + [Gate("CNOT", (2, 3)), _rows((3,), src),
                                                                 Gate("CZ", (3, 6)), _rows((2,), src)]
    for src in itertools.product(range(4), repeat=4):
        yield 3, [Gate("H", (2,)), Gate("RY", (0,), 0.9), Gate("CNOT", (2, 1)), _rows((0, 2), src)]


def _worst(mode, dtype):
    worst = 0.0
    for n, gates in _circuits():
        plan = B.Plan(n, dtype, gates, {"mode": mode})
        got = np.eye(1 << n, dtype=np.complex128)
        for q, m, _ in plan.export():
            got = full_matrix(m, q, n) @ got
        plan.close()
        # entries of every partial product stay below sqrt(2) per repeated
        # row, so the rounding of a gate stays below 32 units
        bound = 32 * EPS * len(gates)
        worst = max(worst, np.abs(got - so.circuit_unitary(gates, n)).max() / bound)
    return worst


def _child(mode, dtype, out):
    out.put(_worst(mode, dtype))


@pytest.mark.parametrize("mode", ["sweep", "auto", "matrix", "pass"])
@pytest.mark.parametrize("dtype", ["c64", "c128"])
def test_every_row_map(mode, dtype):
    """In a process of its own, with a time limit: a planner that follows the
    cycles of a map that has none would not return."""
    ctx = mp.get_context("fork")
    out = ctx.Queue()
    p = ctx.Process(target=_child, args=(mode, dtype, out), daemon=True)
    p.start()
    try:
        worst = out.get(timeout=TIME_LIMIT)
    except Exception:
        worst = None
    p.join(5.0)
    if p.is_alive():
        p.kill()
        p.join()
    assert worst is not None, "the planner did not return"
    assert worst <= 1.0
