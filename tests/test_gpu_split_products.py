"""Register parts and matrix passes of complex64 states on the bf16 matrix
cores: FP32 operands split into three bf16 parts (the top 8 bits, the next 8,
the rest), six part products summed in FP32."""
import numpy as np
import pytest

import oracle
from svgen import Gate, gaussian_state_np, haar_unitary, qft_circuit
from tests.gpu_util import max_err, to_device, to_host

pytestmark = pytest.mark.gpu

# Bound of one 32 x 32 product, elementwise and relative to sum_j |u_ij||x_j|:
# the matrix entry is rounded to FP32 (2^-24); of each real product the dropped
# parts are below 2^-24; the 2 x 6 x 32 part products of a real or imaginary
# part are accumulated in FP32, at most 2 roundings of 2^-24 per matrix
# instruction (24 of them) and the difference of two sums; complex: sqrt(2).
PRODUCT_TOL = (1 + 1 + 2 * 24 + 2) * 2.0 ** -24 * np.sqrt(2.0)


@pytest.fixture(scope="module")
def sv():
    import paper_2409_14697_amd as sv
    return sv


def one_stage(sv, n, qubits, u, psi):
    """Apply u twice-fused: two gates on the same tile make one matrix pass of two
    stages (the second is the identity, exact in the split)."""
    gates = [Gate("MATRIX", qubits, matrix=u), Gate("MATRIX", tuple(reversed(qubits)), matrix=np.eye(32))]
    plan = sv.Plan(n, "c64", gates, {"mode": "matrix", "max_fuse_qubits": 0})
    assert [k for k, _, _ in plan.passes()] == [4]
    t, host_in = to_device(psi, "c64")
    st = sv.StateVector(n, "c64", tensor=t, init=False)
    st.apply_plan(plan)
    st.sync()
    out = to_host(t)
    st.close()
    plan.close()
    return out, host_in


# one column block per wave (12), two (13), several tiles (15); members on
# local bit 0 (16-byte LDS slots) or not
@pytest.mark.parametrize("n", [12, 13, 15])
@pytest.mark.parametrize("qubits", [(0, 1, 2, 3, 4), (7, 0, 11, 3, 9), (5, 1, 8, 2, 10), (11, 10, 9, 8, 7)])
def test_product_error_over_the_exponent_range(sv, n, qubits):
    """Amplitudes from 1 down to 2^-60 in the same columns: every output is
    within the FP32 bound of its own terms, so small ones keep their digits."""
    rng = np.random.default_rng(n)
    u = haar_unitary(32, rng)
    psi = gaussian_state_np(n, 3) * np.exp2(-60.0 * rng.random(1 << n))
    out, host_in = one_stage(sv, n, qubits, u, psi)
    ref = oracle.run([Gate("MATRIX", qubits, matrix=u)], psi0=host_in)
    terms = oracle.run([Gate("MATRIX", qubits, matrix=np.abs(u).astype(np.complex128))],
                       psi0=np.abs(host_in).astype(np.complex128)).real
    assert np.max(np.abs(out - ref) / terms) <= PRODUCT_TOL


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_not_finite_stays_in_its_group(sv, value):
    n, qubits = 13, (2, 5, 0, 9, 12)
    u = haar_unitary(32, np.random.default_rng(5))
    psi = gaussian_state_np(n, 4)
    bad = 1234
    host = psi.astype(np.complex64)
    host[bad] = complex(value, 0.0)
    out, _ = one_stage(sv, n, qubits, u, host.astype(np.complex128))
    mask = sum(1 << q for q in qubits)
    group = (np.arange(1 << n) & ~mask) == (bad & ~mask)
    assert not np.any(np.isfinite(out[group].real) & np.isfinite(out[group].imag))
    assert np.all(np.isfinite(out[~group]))
    host[bad] = 0
    ref = oracle.run([Gate("MATRIX", qubits, matrix=u)], psi0=host.astype(np.complex128))
    assert max_err(out[~group], ref[~group]) <= 1e-6


@pytest.mark.parametrize("n,lds", [(6, 0), (8, 0), (11, 6), (12, 0), (13, 9), (14, 13), (16, 12)])
def test_tile_stages_as_matrices(sv, n, lds):
    """Stages whose layers run as one matrix, with lane items, factors of the
    register index and store maps around them (QFT blocks), full and small
    tiles; the same circuit without the matrix cores."""
    gates = qft_circuit(n) + [Gate("RY", (q,), 0.3 + q) for q in range(n)] + qft_circuit(n)
    psi = gaussian_state_np(n, 8)
    outs = []
    for mfma in (1, 0):
        t, host_in = to_device(psi, "c64")
        st = sv.StateVector(n, "c64", tensor=t, init=False)
        st.apply_circuit(gates, {"mode": "pass", "lds_qubits": lds, "fp32_mfma": mfma})
        st.sync()
        outs.append(to_host(t))
        st.close()
    ref = oracle.run(gates, psi0=host_in)
    assert max_err(outs[0], ref) <= 1e-5 and max_err(outs[1], ref) <= 1e-5


def test_batched_steps_of_every_variant(sv):
    """States whose passes need different kernel variants in one step: bitwise
    the plans applied alone."""
    specs = [(13, qft_circuit(13), {"mode": "pass"}), (14, [Gate("RY", (q,), 0.1 * q) for q in range(14)], {"mode": "pass"}),
             (13, [Gate("MATRIX", (q, 7, 12, 3, 9), matrix=haar_unitary(32, np.random.default_rng(q))) for q in (1, 2, 4)],
              {"mode": "matrix", "max_fuse_qubits": 0})]
    states, programs, alone = [], [], []
    for i, (n, gates, opts) in enumerate(specs):
        plan = sv.Plan(n, "c64", gates, opts)
        t, _ = to_device(gaussian_state_np(n, i), "c64")
        s = sv.StateVector(n, "c64", tensor=t, init=False)
        s.apply_plan(plan)
        s.sync()
        alone.append(to_host(t))
        t2, _ = to_device(gaussian_state_np(n, i), "c64")
        states.append(sv.StateVector(n, "c64", tensor=t2, init=False))
        programs.append(sv.Program(plan))
    b = sv.Batcher()
    for k in range(max(p.n_passes for p in programs)):
        act = [i for i, p in enumerate(programs) if k < p.n_passes]
        b.run([states[i] for i in act], [programs[i] for i in act], [k] * len(act))
    for s, a in zip(states, alone):
        s.sync()
        assert np.array_equal(to_host(s.tensor), a)
