"""Plans of complex64 states that renormalise: a rescale comes at the end of the
pass that completes an interval, so matrix passes stay short."""
import numpy as np
import pytest

from paper_2409_14697_amd import binding as B
from svgen import Gate, haar_unitary

MATRIX_PASS = 4
PASS_OPS = 10  # ops of a matrix pass in such a plan, at most


@pytest.mark.parametrize("interval", [0, 1, 2, 10, 25])
@pytest.mark.parametrize("mode", ["matrix", "auto"])
@pytest.mark.parametrize("n", [12, 13])
def test_matrix_passes_stay_short(interval, mode, n):
    rng = np.random.default_rng(n)
    gates = [Gate("MATRIX", tuple(int(q) for q in rng.choice(n, 5, replace=False)), matrix=haar_unitary(32, rng))
             for _ in range(90)]
    plan = B.Plan(n, "c64", gates, {"mode": mode, "max_fuse_qubits": 0, "renorm_interval": interval})
    ops = [k for kind, k, _ in plan.passes() if kind == MATRIX_PASS]
    assert sum(ops) == 90
    assert max(ops) == PASS_OPS if interval else max(ops) > PASS_OPS
