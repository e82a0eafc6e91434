"""Matrix stages of complex64 states over the whole FP32 range: small amplitudes
and matrix entries keep their digits, and large ones stay finite."""
import numpy as np
import pytest

import oracle
from svgen import Gate, gaussian_state_np, haar_unitary
from tests.test_gpu_split_tiles import layers, run, tile_plans

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -24
TINY = 2.0 ** -149  # the spacing of FP32 below 2^-126
# One 32 x 32 product, elementwise and relative to sum_j |u_ij||x_j|: the
# matrix entry is rounded to FP32 (1 unit); the operands' parts after the top
# one are below 2^-7 and 2^-16 of an amplitude and 2^-8 and 2^-17 of an entry,
# so each of the three dropped part products is at most 2^-24 and their sum
# 2^-23 (2 units); a real or an imaginary part takes 24 matrix instructions of
# at most 2 roundings of the sum and a difference (50 units); complex: sqrt(2).
PRODUCT_TOL = (1 + 2 + 50) * EPS * np.sqrt(2.0)
QUBITS = [(0, 1, 2, 3, 4), (5, 1, 8, 2, 10)]  # members on local bit 0 first, or not


@pytest.fixture(scope="module")
def sv():
    import paper_2409_14697_amd as sv
    return sv


def matrix_pass(sv, n, qubits, u, psi, first=True):
    """One matrix pass of u and of the identity, which changes nothing."""
    gates = [Gate("MATRIX", qubits, matrix=u), Gate("MATRIX", tuple(reversed(qubits)), matrix=np.eye(32))]
    if not first:
        gates.reverse()
    opts = {"mode": "matrix", "max_fuse_qubits": 0}
    plan = sv.Plan(n, "c64", gates, opts)
    assert [k for k, _, _ in plan.passes()] == [4]
    plan.close()
    return run(sv, n, gates, psi, opts)


def check_product(out, host_in, qubits, u):
    ref = oracle.run([Gate("MATRIX", qubits, matrix=u)], psi0=host_in)
    terms = oracle.run([Gate("MATRIX", qubits, matrix=np.abs(u).astype(np.complex128))],
                       psi0=np.abs(host_in).astype(np.complex128)).real
    assert np.all(np.abs(out - ref) <= PRODUCT_TOL * terms + TINY)


@pytest.mark.parametrize("n", [12, 13])
@pytest.mark.parametrize("qubits", QUBITS)
@pytest.mark.parametrize("low,high", [(-148, -100), (-126, -118), (-148, 0), (-60, 30), (-100, 90), (85, 100), (100, 120)])
def test_amplitudes_of_every_size(sv, n, qubits, low, high):
    """Magnitudes spread between 2^low and 2^high, subnormal ones among them."""
    rng = np.random.default_rng(n)
    e = low + (high - low) * rng.random(1 << n)
    psi = np.exp2(e) * np.exp(2j * np.pi * rng.random(1 << n))
    u = haar_unitary(32, rng)
    out, host_in = matrix_pass(sv, n, qubits, u, psi)
    assert np.all(np.isfinite(out))
    check_product(out, host_in, qubits, u)


@pytest.mark.parametrize("n", [12, 13])
@pytest.mark.parametrize("qubits", QUBITS)
def test_small_amplitudes_beside_large_ones(sv, n, qubits):
    """A matrix that leaves the lower half of its members to themselves: theirs
    are 2^-120, the others 1 (and 2^60)."""
    rng = np.random.default_rng(3)
    u = np.zeros((32, 32), np.complex128)
    u[:16, :16] = haar_unitary(16, rng)
    u[16:, 16:] = haar_unitary(16, rng)
    for big in (1.0, 2.0 ** 60):
        psi = gaussian_state_np(n, 5) * 64.0
        low = (np.arange(1 << n) >> qubits[0]) & 1 == 1  # qubits[0]: the most significant member bit
        psi = np.where(low, psi * 2.0 ** -120, psi * big)
        out, host_in = matrix_pass(sv, n, qubits, u, psi)
        check_product(out, host_in, qubits, u)


@pytest.mark.parametrize("n", [12, 13])
@pytest.mark.parametrize("scale", [-120, -100, 30, 50, 100])
@pytest.mark.parametrize("first", [True, False])
def test_matrix_entries_of_every_size(sv, n, scale, first):
    rng = np.random.default_rng(6)
    u = haar_unitary(32, rng) * np.exp2(-6.0 * rng.random((32, 32)) + scale)
    out, host_in = matrix_pass(sv, n, QUBITS[1], u, gaussian_state_np(n, 7) * (2.0 ** 10), first)
    assert np.all(np.isfinite(out))
    check_product(out, host_in, QUBITS[1], u)


@pytest.mark.parametrize("n,lds", [(6, 0), (9, 0), (12, 9), (13, 0), (15, 13)])
@pytest.mark.parametrize("scale", [-122, -105, 60, 100, 115])
def test_tile_stages_of_every_size(sv, n, lds, scale):
    """As at ordinary magnitudes (the tests of the tile stages)."""
    gates = layers(n, 3, seed=n)
    opts, stages, matrix_stages = tile_plans(sv, n, gates, lds)
    assert matrix_stages >= 3  # (a tail of few gates may stay on the VALU)
    psi = gaussian_state_np(n, 8) * np.exp2(0.5 * n + scale)
    for o in opts:
        out, host_in = run(sv, n, gates, psi, o)
        ref = oracle.run(gates, psi0=host_in)
        err = np.linalg.norm(out - ref) / np.linalg.norm(ref)
        assert err <= 4 * stages * EPS + TINY * np.sqrt(2.0 ** n * stages) / np.linalg.norm(ref)


@pytest.mark.parametrize("n", [6, 9, 13])
def test_products_of_small_entries(sv, n):
    """Five gates with diagonal entries of 2^-25: the stage's matrix has entries
    down to 2^-125, and from one amplitude per group its results."""
    rng = np.random.default_rng(2)
    small = np.diag([2.0 ** -25, 2.0 ** -25]) + np.array([[0, 1], [1, 0]])
    gates = [Gate("MATRIX", (q,), matrix=haar_unitary(2, rng) * small) for q in range(5)]
    opts, _, matrix_stages = tile_plans(sv, n, gates, 0)
    assert matrix_stages == 1
    psi = np.where(np.arange(1 << n) & 31, 0.0, gaussian_state_np(n, 3) * np.exp2(0.5 * n))
    for o in opts:
        out, host_in = run(sv, n, gates, psi, o)
        ref = oracle.run(gates, psi0=host_in)
        # one term per result; each gate rounds its entry and its product, and
        # underflow adds one spacing per gate
        assert np.all(np.abs(out - ref) <= PRODUCT_TOL * np.abs(ref) + 5 * TINY)
