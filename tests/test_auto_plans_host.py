"""What the automatic plan of a complex64 state is made of: matrix passes pay for
the build of their operands, a launch of its own that few gates on a small
state do not earn."""
import numpy as np
import pytest

from paper_2409_14697_amd import binding as B
from svgen import Gate, brickwork_circuit, haar_unitary

TILE_PASS, MATRIX_PASS = 1, 4


def kinds(n, gates):
    plan = B.Plan(n, "c64", gates)
    return [k for k, _, _ in plan.passes()]


@pytest.mark.parametrize("n", [12, 13, 16, 20])
def test_few_gates_on_small_states(n):
    """A few microseconds either way: a tile pass and a sweep, not a matrix pass."""
    u = haar_unitary(8, np.random.default_rng(1))
    gates = [Gate("P", (4,), 0.4), Gate("MATRIX", (6, 11, 3), matrix=u), Gate("X", (5,))]
    assert MATRIX_PASS not in kinds(n, gates)


@pytest.mark.parametrize("n", [12, 14, 20, 25])
def test_deep_circuits(n):
    """Layers of rotations and CNOTs stay in matrix passes, small states too."""
    assert MATRIX_PASS in kinds(n, brickwork_circuit(n, 10, seed=n))
