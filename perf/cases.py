"""The work a user of this simulator has it do, as measurable cases.

A case names a kind of call and its sizes:

  gates    single gates, one call each (StateVector.apply_gate): every kind of
           the gate benchmark on targets spread over the index, or the
           N=16, 200-gate layered circuit run gate by gate
  plan     a circuit planned once and applied to a state (apply_plan)
  apply    the whole call with a new circuit: start state, planning,
           execution and the marginal of the lowest qubits (apply_circuit)
  serve    a closed loop of circuit requests through the batching server
  readout  marginals, the norm and a qubit reordering of a state

Circuits follow the recipes of the benchmark program: layered (random
rotations and a random CNOT matching), brickwork, QFT, complete-graph QAOA
and Haar-random fused gates.  States are normalised complex Gaussians where a
circuit acts on an arbitrary state (QFT, fused gates, single gates, readout)
and |0..0> where a program simulates a circuit from its start.
"""
import math
from collections import namedtuple

import numpy as np
import torch

import paper_2409_14697_amd as sv
from paper_2409_14697_amd import binding, serve

Gate = namedtuple("Gate", "kind qubits theta matrix", defaults=(0.0, None))

BYTES = {"c64": 8, "c128": 16}
TORCH = {"c64": torch.complex64, "c128": torch.complex128}
KINDS = ("H", "X", "RZ", "CNOT", "CZ", "SWAP", "CPHASE")


def listed():
    return [
        # a variational or sampling loop on a small register: the plan is kept,
        # launches and latency are all there is
        {"name": "plan_layered_n12_c64", "call": "plan", "circuit": "layered", "n": 12, "depth": 20, "dtype": "c64",
         "start": True},
        # an interactive session: 200 gates one call each (the N=16 layered circuit)
        {"name": "gates_layered_n16_c128", "call": "gates", "circuit": "layered", "n": 16, "depth": 9, "dtype": "c128"},
        # a circuit seen once: planning counts
        {"name": "apply_layered_n20_c64", "call": "apply", "circuit": "layered", "n": 20, "depth": 10, "dtype": "c64"},
        # the gate benchmark: every kind of gate on low, middle and high targets
        {"name": "gates_sweep_n28_c128", "call": "gates", "circuit": "sweep", "n": 28, "depth": 6, "dtype": "c128"},
        # the transform at the heart of phase estimation, on an arbitrary state
        {"name": "plan_qft_n28_c64", "call": "plan", "circuit": "qft", "n": 28, "depth": 1, "dtype": "c64",
         "start": False},
        # optimisation circuits in double precision: long runs of phase gates
        {"name": "plan_qaoa_n27_c128", "call": "plan", "circuit": "qaoa", "n": 27, "depth": 5, "dtype": "c128",
         "start": True},
        # deep random circuits, the largest case, single precision
        {"name": "plan_brickwork_n30_c64", "call": "plan", "circuit": "brickwork", "n": 30, "depth": 20,
         "dtype": "c64", "start": True},
        # the same family in double precision, an odd and smaller register
        {"name": "plan_brickwork_n25_c128", "call": "plan", "circuit": "brickwork", "n": 25, "depth": 20,
         "dtype": "c128", "start": True},
        # user-supplied dense unitaries on random qubits (the precision form's gates)
        {"name": "plan_haar_n28_c64", "call": "plan", "circuit": "haar", "n": 28, "depth": 12, "dtype": "c64",
         "start": False},
        {"name": "plan_haar_n27_c128", "call": "plan", "circuit": "haar", "n": 27, "depth": 12, "dtype": "c128",
         "start": False},
        # a serving process: many requests of different sizes in flight at once
        {"name": "serve_48_c64", "call": "serve", "circuit": "layered", "n": 24, "depth": 40, "dtype": "c64",
         "requests": 48},
        # what follows a simulation: sampling marginals, checking the norm, reordering
        {"name": "readout_n29_c64", "call": "readout", "circuit": "", "n": 29, "depth": 0, "dtype": "c64"},
    ]


def draw(rng):
    """One more case of the same ranges; its state and gate count stay at or
    below those of the largest listed case of its kind."""
    dtype = rng.choice(("c64", "c128"))
    less = 1 if dtype == "c128" else 0  # the same bytes
    kind = rng.choice(("gates", "sweep", "layered", "apply", "qft", "qaoa", "brickwork", "haar", "serve", "readout"))
    if kind == "gates":
        return {"call": "gates", "circuit": "layered", "n": rng.randint(10, 18), "depth": rng.randint(4, 9),
                "dtype": dtype}
    if kind == "sweep":
        return {"call": "gates", "circuit": "sweep", "n": rng.randint(18, 29 - less), "depth": rng.randint(3, 6),
                "dtype": dtype}
    if kind == "layered":
        return {"call": "plan", "circuit": "layered", "n": rng.randint(8, 24), "depth": rng.randint(5, 20),
                "dtype": dtype, "start": True}
    if kind == "apply":
        return {"call": "apply", "circuit": "layered", "n": rng.randint(10, 22), "depth": rng.randint(4, 12),
                "dtype": dtype}
    if kind == "qft":
        return {"call": "plan", "circuit": "qft", "n": rng.randint(16, 29 - less), "depth": 1, "dtype": dtype,
                "start": False}
    if kind == "qaoa":
        return {"call": "plan", "circuit": "qaoa", "n": rng.randint(14, 28 - less), "depth": rng.randint(1, 5),
                "dtype": dtype, "start": True}
    if kind == "brickwork":
        return {"call": "plan", "circuit": "brickwork", "n": rng.randint(16, 28 - less), "depth": rng.randint(6, 20),
                "dtype": dtype, "start": True}
    if kind == "haar":
        return {"call": "plan", "circuit": "haar", "n": rng.randint(16, 28 - less), "depth": rng.randint(4, 12),
                "dtype": dtype, "start": False}
    if kind == "serve":
        return {"call": "serve", "circuit": "layered", "n": rng.randint(18, 23), "depth": rng.randint(12, 40),
                "dtype": dtype, "requests": rng.randint(8, 48)}
    return {"call": "readout", "circuit": "", "n": rng.randint(14, 29 - less), "depth": 0, "dtype": dtype}


# ------------------------------------------------------------------ circuits
def _haar(d, rng):
    z = rng.standard_normal((d, d)) + 1j * rng.standard_normal((d, d))
    q, r = np.linalg.qr(z)
    return q * (np.diag(r) / np.abs(np.diag(r)))[np.newaxis, :]


def _circuit(circuit, n, depth, rng):
    gates = []
    if circuit == "layered":
        for _ in range(depth):
            for q in range(n):
                kind = ("H", "RX", "RY", "RZ")[int(rng.integers(4))]
                gates.append(Gate(kind, (q,), 0.0 if kind == "H" else float(rng.uniform(0.0, 2.0 * math.pi))))
            p = [int(x) for x in rng.permutation(n)]
            gates += [Gate("CNOT", (p[2 * m], p[2 * m + 1])) for m in range(n // 2)]
    elif circuit == "brickwork":
        for layer in range(depth):
            for q in range(n):
                gates.append(Gate(("RX", "RY", "RZ")[int(rng.integers(3))], (q,), float(rng.uniform(0.0, 2.0 * math.pi))))
            gates += [Gate("CNOT", (a, a + 1)) for a in range(layer % 2, n - 1, 2)]
    elif circuit == "qft":
        for j in range(n - 1, -1, -1):
            gates.append(Gate("H", (j,)))
            gates += [Gate("CPHASE", (k, j), math.pi / float(1 << (j - k))) for k in range(j - 1, -1, -1)]
        gates += [Gate("SWAP", (q, n - 1 - q)) for q in range(n // 2)]
    elif circuit == "qaoa":
        gates += [Gate("H", (q,)) for q in range(n)]
        for _ in range(depth):
            gamma, beta = float(rng.uniform(0.0, math.pi)), float(rng.uniform(0.0, 0.5 * math.pi))
            gates += [Gate("RZZ", (a, b), gamma) for a in range(n) for b in range(a + 1, n)]
            gates += [Gate("RX", (q,), 2.0 * beta) for q in range(n)]
    elif circuit == "haar":  # fused gates of 3 to 6 qubits on ordered random sets
        for g in range(depth):
            k = (5, 6, 4, 6, 5, 3)[g % 6]
            gates.append(Gate("MATRIX", tuple(int(x) for x in rng.choice(n, k, replace=False)), 0.0, _haar(1 << k, rng)))
    elif circuit == "sweep":  # every kind on `depth` targets spread over the index
        for kind in KINDS:
            for t in sorted({round(i * (n - 1) / (depth - 1)) for i in range(depth)}):
                theta = float(rng.uniform(0.0, 2.0 * math.pi)) if kind in ("RZ", "CPHASE") else 0.0
                if kind in ("H", "X", "RZ"):
                    gates.append(Gate(kind, (t,), theta))
                    continue
                p = int(rng.integers(n - 1))
                p += p >= t
                gates.append(Gate(kind, (p, t) if kind == "CNOT" else (t, p), theta))
    return gates


def _requests(case, seed):
    """(n, gates) of every request: n from 12 up, `depth` layer pairs at most;
    the sizes belong to the case, the gates to the seed."""
    sizes, rng = np.random.default_rng([case["n"], case["depth"], 4]), np.random.default_rng([seed, 5])
    out = []
    for _ in range(case["requests"]):
        n = int(sizes.integers(12, case["n"] + 1))
        out.append((n, _circuit("layered", n, int(sizes.integers(case["depth"] // 4, case["depth"] + 1)), rng)))
    return out


def _gaussian(n, dtype, seed, device):
    g = torch.Generator(device=device)
    g.manual_seed(seed)
    t = torch.empty(1 << n, dtype=TORCH[dtype], device=device)
    parts = torch.view_as_real(t)
    parts.normal_(generator=g)
    parts.mul_(2.0 ** (-0.5 * (n + 1)))  # unit norm up to the draw's own deviation
    return t


def _readout(case, seed):
    """Qubit lists of the marginals, and a qubit reordering."""
    n = case["n"]
    rng = np.random.default_rng([seed, 6])
    k = min(n, 10)
    return (list(range(min(n, 16) - 1, -1, -1)), [int(x) for x in rng.choice(n, k, replace=False)],
            list(range(n - 1, n - 1 - k, -1)), [int(x) for x in rng.permutation(n)])


# ------------------------------------------------------------------- calls
def prepare(case, seed):
    n, dtype, call = case["n"], case["dtype"], case["call"]
    st = {"case": case}
    if call == "serve":
        reqs = _requests(case, seed)
        st["jobs"] = [(m, binding.make_gates(g), len(g)) for m, g in reqs]
        st["engine"] = serve.DeviceEngine(dtype)
        return st
    st["state"] = sv.StateVector(n, dtype, tensor=_gaussian(n, dtype, seed, "cuda"), init=False)
    if call == "readout":
        st["low"], st["some"], st["high"], st["dest"] = _readout(case, seed)
        st["out"] = [torch.empty(1 << len(q), dtype=torch.float64, device="cuda")
                     for q in (st["low"], st["some"], st["high"], [])]
        return st
    gates = _circuit(case["circuit"], n, case["depth"], np.random.default_rng([seed, 1]))
    if call == "plan":
        st["plan"] = sv.Plan(n, dtype, gates)
    else:
        st["gates"] = gates
    if call == "apply":
        st["probs"] = torch.empty(1 << min(n, 10), dtype=torch.float64, device="cuda")
    return st


def _carried(case, probs):
    """A circuit's marginals as a client keeps them: in the precision that the
    simulated state carries (the library sums them in FP64)."""
    if case["dtype"] == "c128":
        return probs
    return probs.float() if isinstance(probs, torch.Tensor) else probs.astype(np.float32)


def run(st):
    case = st["case"]
    call = case["call"]
    if call == "serve":
        jobs = [serve.Job(rid=i, n=n, arrival=0.0, gates=g, n_gates=c) for i, (n, g, c) in enumerate(st["jobs"])]
        serve.Server(st["engine"], budget_bytes=64 << 30, plan_workers=8).run(jobs)
        return [_carried(case, j.probs) for j in jobs]
    s = st["state"]
    if call == "gates":
        for g in st["gates"]:
            s.apply_gate(g)
        return s.tensor
    if call == "plan":
        if case["start"]:
            s.init_basis(0)
        s.apply_plan(st["plan"])
        return s.tensor
    if call == "apply":
        s.init_basis(0)
        s.apply_circuit(st["gates"])
        probs = s.measure_probs(list(range(min(case["n"], 10) - 1, -1, -1)), out=st["probs"])
        return s.tensor, _carried(case, probs)
    for q, out in zip((st["low"], st["some"], st["high"], []), st["out"]):
        s.measure_probs(q, out=out)
    s.permute_qubits(st["dest"])
    return s.tensor, st["out"]


# -------------------------------------------------------------------- work
def _flops(gates, n):
    """Real operations of the gates: a complex product is 6, a sum 2; a run of
    phase gates is one product for each amplitude."""
    per, phases = 0.0, False
    for g in gates:
        if g.kind in ("RZ", "RZZ", "CPHASE"):
            if not phases:
                per += 6.0
            phases = True
            continue
        if g.kind in ("X", "CNOT", "SWAP", "CZ"):
            continue
        phases = False
        if g.kind == "MATRIX":
            per += 8.0 * (1 << len(g.qubits)) - 2.0
        else:  # H, RX, RY: two products by real (or imaginary) numbers and a sum
            per += 6.0
    return per * float(1 << n)


def work(case):
    n, call = case["n"], case["call"]
    size = float(BYTES[case["dtype"]] << n)
    if call == "serve":
        b = f = 0.0
        for m, gates in _requests(case, 0):
            b += float(BYTES[case["dtype"]] << m) + float(8 << min(m, 16))
            f += _flops(gates, m)
        return {"bytes": b, "flops": f}
    if call == "readout":
        # the marginals share one read; the reordering reads and writes
        return {"bytes": 3.0 * size, "flops": 4 * 4.0 * (1 << n)}
    gates = _circuit(case["circuit"], n, case["depth"], np.random.default_rng([0, 1]))
    if call == "gates":
        # every call reads and writes what its gate changes
        part = {"CNOT": 0.5, "CZ": 0.25, "SWAP": 0.5, "CPHASE": 0.25}
        return {"bytes": sum(2.0 * size * part.get(g.kind, 1.0) for g in gates), "flops": _flops(gates, n)}
    read = 0.0 if call == "apply" or case.get("start") else size
    more = size if call == "apply" else 0.0  # the marginal reads the result
    return {"bytes": read + size + more, "flops": _flops(gates, n)}


# ------------------------------------------------------------------- exact
def _matrix(g):
    t = g.theta
    c, s = math.cos(0.5 * t), math.sin(0.5 * t)
    r = math.sqrt(0.5)
    return {"H": [[r, r], [r, -r]], "X": [[0, 1], [1, 0]], "RX": [[c, -1j * s], [-1j * s, c]],
            "RY": [[c, -s], [s, c]]}[g.kind]


def _phases(g):
    """Diagonal entries in local order, for the diagonal kinds."""
    e = lambda a: complex(math.cos(a), math.sin(a))  # noqa: E731
    return {"RZ": lambda t: (e(-0.5 * t), e(0.5 * t)), "RZZ": lambda t: (e(-0.5 * t), e(0.5 * t), e(0.5 * t), e(-0.5 * t)),
            "CZ": lambda t: (1, 1, 1, -1), "CPHASE": lambda t: (1, 1, 1, e(t))}[g.kind](g.theta)


def _split(psi, n, qubits):
    """A view of the state with one axis for each qubit, in their order, and
    the others around them."""
    order = sorted(qubits, reverse=True)
    dims, top = [], n
    for q in order:
        dims += [1 << (top - 1 - q), 2]
        top = q
    dims.append(1 << top)
    axis = {q: 2 * i + 1 for i, q in enumerate(order)}
    rest = [a for a in range(len(dims)) if a % 2 == 0]
    return psi.view(dims).permute([axis[q] for q in qubits] + rest)


def _apply(psi, n, g):
    v = _split(psi, n, g.qubits)
    k = len(g.qubits)
    if g.kind == "MATRIX":
        u = torch.from_numpy(np.ascontiguousarray(g.matrix)).to(psi.device)
        y = u @ v.contiguous().view(1 << k, -1)
        v.copy_(y.view(v.shape))
    elif g.kind == "CNOT":
        x = v[1, 0].clone()
        v[1, 0].copy_(v[1, 1])
        v[1, 1].copy_(x)
    elif g.kind == "SWAP":
        x = v[0, 1].clone()
        v[0, 1].copy_(v[1, 0])
        v[1, 0].copy_(x)
    elif k == 1 and g.kind != "RZ":
        (a, b), (c, d) = _matrix(g)
        x, y = v[0].clone(), v[1]
        v[0].mul_(a).add_(y, alpha=b)
        y.mul_(d).add_(x, alpha=c)
    else:
        for i, f in enumerate(_phases(g)):
            if f != 1:
                (v[i] if k == 1 else v[i >> 1, i & 1]).mul_(f)


def _probs(psi, n, qubits):
    p = torch.view_as_real(psi).square().sum(-1)
    for q in range(n - 1, -1, -1):  # sum over the other qubits, one run of them at a time
        if q not in qubits and (q == n - 1 or q + 1 in qubits):
            low = q
            while low > 0 and low - 1 not in qubits:
                low -= 1
            above = sum(1 for x in qubits if x > q)
            p = p.reshape(1 << above, 1 << (q - low + 1), 1 << low).sum(1)
    order = sorted(qubits, reverse=True)
    p = p.reshape([2] * len(qubits)).cpu().numpy().transpose([order.index(q) for q in qubits])
    return torch.from_numpy(np.ascontiguousarray(p).reshape(-1))


def _zero(n, device):
    psi = torch.zeros(1 << n, dtype=torch.complex128, device=device)
    psi[0] = 1
    return psi


def exact(case, seed):
    n, call = case["n"], case["call"]
    device = "cuda"
    if call == "serve":
        out = []
        for m, gates in _requests(case, seed):
            psi = _zero(m, device)
            for g in gates:
                _apply(psi, m, g)
            out.append(_probs(psi, m, list(range(min(m, 16) - 1, -1, -1))).numpy())
        return out
    psi = _gaussian(n, case["dtype"], seed, device).to(torch.complex128)
    if call == "readout":
        low, some, high, dest = _readout(case, seed)
        probs = [_probs(psi, n, q) for q in (low, some, high, [])]
        # qubit q moves to bit dest[q]
        inverse = [0] * n
        for q, p in enumerate(dest):
            inverse[p] = q
        moved = psi
        cur = list(range(n))  # cur[p]: the qubit now at bit p
        for p in range(n):
            j = cur.index(inverse[p])
            if j != p:
                _apply(moved, n, Gate("SWAP", (p, j)))
                cur[p], cur[j] = cur[j], cur[p]
        return moved, probs
    if call == "apply" or case.get("start"):
        psi = _zero(n, device)
    for g in _circuit(case["circuit"], n, case["depth"], np.random.default_rng([seed, 1])):
        _apply(psi, n, g)
    if call == "apply":
        return psi, _probs(psi, n, list(range(min(n, 10) - 1, -1, -1)))
    return psi
