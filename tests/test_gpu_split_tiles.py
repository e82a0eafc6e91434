"""Register parts of tile stages as matrices on the bf16 matrix cores (complex64):
which stages run so, the digits of their results, and values that are not
finite."""
import numpy as np
import pytest

import oracle
from svgen import (Gate, brickwork_circuit, gaussian_state_np, haar_unitary, layered_circuit, qaoa_circuit,
                   qft_circuit)
from tests.gpu_util import to_device, to_host

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -24
TINY = 2.0 ** -149               # the spacing of FP32 below 2^-126
FRAGMENTS = 32 * 32 * 2 * 3 * 2  # device bytes of one stage's operands


@pytest.fixture(scope="module")
def sv():
    import paper_2409_14697_amd as sv
    return sv


def run(sv, n, gates, psi, opts):
    plan = sv.Plan(n, "c64", gates, opts)
    t, host_in = to_device(psi, "c64")
    st = sv.StateVector(n, "c64", tensor=t, init=False)
    st.apply_plan(plan)
    st.sync()
    out = to_host(t)
    st.close()
    plan.close()
    return out, host_in


def layers(n, reps, seed, qubits=None):
    """Dense single-qubit gates, CNOTs between their layers: stages without lane
    items, whose register part is one matrix."""
    rng = np.random.default_rng(seed)
    gates = []
    for r in range(reps):
        gates += [Gate("MATRIX", (q,), matrix=haar_unitary(2, rng)) for q in (qubits or range(n))]
        if r + 1 < reps:
            gates += [Gate("CNOT", (q, (q + 1 + r) % n)) for q in range(0, n - 1, 2)]
    return gates


def tile_plans(sv, n, gates, lds):
    """Options with and without the matrix cores, and the number of stages; the
    plans differ in the operands of the stages that run as matrices."""
    opts = [{"mode": "pass", "lds_qubits": lds, "fp32_mfma": m} for m in (1, 0)]
    plans = [sv.Plan(n, "c64", gates, o) for o in opts]
    stages = [sum(s for _, _, _, s in p.passes(stages=True)) for p in plans]
    extra = plans[0].program_bytes() - plans[1].program_bytes()
    for p in plans:
        p.close()
    assert stages[0] == stages[1]
    return opts, stages[0], extra // FRAGMENTS


@pytest.mark.parametrize("n,lds", [(6, 0), (9, 0), (12, 9), (13, 0), (15, 13)])
@pytest.mark.parametrize("scale", [0, -40, 20])
def test_tile_stages_keep_every_digit(sv, n, lds, scale):
    """The error of a stage in the 2-norm: entries rounded once and dropped parts
    below 2^-23 of a product would give 4 units if all errors had one sign;
    their signs are independent, and a missing low part gives about 70."""
    gates = layers(n, 3, seed=n)
    opts, stages, matrix_stages = tile_plans(sv, n, gates, lds)
    assert matrix_stages >= 3  # (a tail of few gates may stay on the VALU)
    psi = gaussian_state_np(n, 8) * np.exp2(0.5 * n + scale)
    for o in opts:
        out, host_in = run(sv, n, gates, psi, o)
        ref = oracle.run(gates, psi0=host_in)
        err = np.linalg.norm(out - ref) / np.linalg.norm(ref)
        assert err <= 4 * stages * EPS + TINY * np.sqrt(2.0 ** n * stages) / np.linalg.norm(ref)


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("n,lds", [(6, 0), (9, 0), (13, 0), (15, 13)])
def test_not_finite_reaches_what_the_gates_mix(sv, n, lds, value):
    """Gates on three qubits: eight amplitudes, with and without the matrix
    cores, although a stage's matrix has 32 members."""
    qubits = (0, 2, 5)
    gates = layers(n, 1, seed=4, qubits=qubits)
    opts, _, matrix_stages = tile_plans(sv, n, gates, lds)
    assert matrix_stages == 1
    bad = 37
    psi = gaussian_state_np(n, 9)
    psi[bad] = complex(value, 0.0)
    mask = sum(1 << q for q in qubits)
    group = (np.arange(1 << n) & ~mask) == (bad & ~mask)
    clean = psi.copy()
    clean[bad] = 0.0
    for o in opts:
        out, _ = run(sv, n, gates, psi, o)
        assert not np.any(np.isfinite(out[group].real) & np.isfinite(out[group].imag))
        assert np.all(np.isfinite(out[~group].real) & np.isfinite(out[~group].imag))
        ref = oracle.run(gates, psi0=clean.astype(np.complex64).astype(np.complex128))
        assert np.max(np.abs(out[~group] - ref[~group])) <= 1e-6


@pytest.mark.parametrize("n,lds", [(8, 0), (10, 0), (13, 0), (13, 9), (15, 0)])
def test_mixed_steps_share_a_launch(sv, n, lds):
    """Passes with and without matrix stages in one step: every state as its plan
    leaves it alone, bit for bit."""
    circuits = [qft_circuit(n), layered_circuit(n, n_gates=6 * n, seed=2), qaoa_circuit(n, 1, seed=3),
                [Gate("X", (0,)), Gate("CNOT", (1, 4)), Gate("SWAP", (2, n - 1))], brickwork_circuit(n, 4, seed=1)]
    states, programs, alone, extra = [], [], [], []
    for i, gates in enumerate(circuits):
        plan = sv.Plan(n, "c64", gates, {"mode": "pass", "lds_qubits": lds})
        extra.append(tile_plans(sv, n, gates, lds)[2])
        for out in (alone, states):
            t, _ = to_device(gaussian_state_np(n, i), "c64")
            s = sv.StateVector(n, "c64", tensor=t, init=False)
            out.append(s)
        alone[-1].apply_plan(plan)
        programs.append(sv.Program(plan))
    assert extra[0] > 0 and extra[1] == 0
    b = sv.Batcher()
    for k in range(max(p.n_passes for p in programs)):
        act = [i for i, p in enumerate(programs) if k < p.n_passes]
        b.run([states[i] for i in act], [programs[i] for i in act], [k] * len(act))
    for s, a in zip(states, alone):
        s.sync()
        a.sync()
        assert np.array_equal(to_host(s.tensor), to_host(a.tensor))
