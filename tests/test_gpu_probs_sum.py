"""The chunk sum of the marginal-probability reduction: few and many bins, few
and thousands of chunks, against the oracle."""
import numpy as np
import pytest

import oracle
from svgen import gaussian_state_np
from tests.gpu_util import to_device

pytestmark = pytest.mark.gpu


# (n, measured qubits): one bin over 1 .. 4096 chunks; bins below, at and above
# a block's 32; few chunks with many bins; measured bits low, high and mixed
@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n,qubits", [(9, []), (12, []), (18, []), (21, []), (20, [3]), (20, [19, 0]), (19, [5, 6, 7, 8, 9]),
                                      (19, [18, 2, 9, 0, 11, 4]), (20, list(range(7, -1, -1))),
                                      (20, list(range(16, 3, -1))), (18, list(range(17, 1, -1)))])
def test_marginal_of_every_chunk_shape(dtype, n, qubits):
    import paper_2409_14697_amd as sv
    t, host = to_device(gaussian_state_np(n, n), dtype)
    st = sv.StateVector(n, dtype, tensor=t, init=False)
    p = st.measure_probs(qubits).cpu().numpy()
    again = st.measure_probs(qubits).cpu().numpy()
    st.close()
    ref = oracle.probs(host, qubits) if qubits else np.array([float(np.sum(np.abs(host) ** 2))])
    # sums of non-negative terms: at most one rounding per term on each side,
    # in practice chunked; 2^n / bins terms of 2^-53 each
    tol = (2 << n) / len(ref) * 2.0 ** -53
    assert np.all(np.abs(p - ref) <= tol * ref)
    assert np.array_equal(p, again)
