"""Performance cases: the work a user of the library has it do, through its public entry points.

A case names a path (``kind``), a size, a precision and a circuit structure; ``prepare`` builds what a program holds
before the call (states, circuits, batches, angles drawn from the seed), ``run`` makes one pass through the public
API and returns every output whole, ``work`` states the bytes and operations the pass cannot do without, and
``exact`` gives the same outputs from plain torch in complex128.

The kinds and what they stand for:

* ``train``    one optimiser step's energy and gradient of a one-circuit ansatz on the fused engine (autograd form)
* ``batch``    energies and gradients of many circuits of mixed sizes in one call (parameter sweeps, ensembles)
* ``forward``  one large circuit run forward on the fused engine: its energy and its final state
* ``gates``    gates applied one call at a time to a large state (interactive simulation, the gate benchmark)
* ``ops``      a circuit applied to a state op by op, with diagonal runs fused, or as dense blocks, then a measurement
* ``adjoint``  energy and gradient with a general Pauli-sum Hamiltonian through the op-by-op adjoint sweep
* ``pauli``    the expectation value of a Heisenberg-chain Hamiltonian on a large state, and the state's norm
* ``dense``    fused 4- to 6-qubit blocks applied to a large state
"""
from __future__ import annotations

import math
import random
from typing import Dict, List, NamedTuple, Optional, Tuple

import numpy as np
import torch

import paper_2508_13615_amd as sv


class Op(NamedTuple):
    gate: str
    controls: Tuple[int, ...] = ()
    targets: Tuple[int, ...] = ()
    pidx: int = -1
    value: float = 0.0
    matrix: Optional[np.ndarray] = None


TORCH = {"c128": torch.complex128, "c64": torch.complex64}
SIZE = {"c128": 16, "c64": 8}


# --------------------------------------------------------------------------
# circuits
# --------------------------------------------------------------------------
def hea(n: int, layers: int) -> Tuple[List[Op], int]:
    """Hardware-efficient ansatz: RY and RZ on every qubit, then a CNOT ladder."""
    ops: List[Op] = []
    for layer in range(layers):
        for q in range(n):
            ops.append(Op("RY", (), (q,), 2 * (layer * n + q)))
            ops.append(Op("RZ", (), (q,), 2 * (layer * n + q) + 1))
        for q in range(n - 1):
            ops.append(Op("X", (q,), (q + 1,)))
    return ops, 2 * n * layers


def qft(n: int) -> Tuple[List[Op], int]:
    """Quantum Fourier transform (no final swaps) of a product state prepared by one rotation per qubit."""
    ops: List[Op] = [Op("RY", (), (q,), q) for q in range(n)]
    for j in range(n - 1, -1, -1):
        ops.append(Op("H", (), (j,)))
        for c in range(j - 1, -1, -1):
            ops.append(Op("PHASE", (c,), (j,), -1, math.pi / float(1 << (j - c))))
    return ops, n


def universal(n: int) -> Tuple[List[Op], int]:
    """Universal circuit (n(n-1) CNOTs and n(n+1) Z rotations) on a product state prepared by one rotation per qubit."""
    ops: List[Op] = [Op("RY", (), (q,), q) for q in range(n)]
    for t in range(n):
        k = 1
        ops.append(Op("RZ", (), (t,), -1, math.pi / 2.0))
        for c in range(n):
            if c == t:
                continue
            k += 1
            ops.append(Op("X", (c,), (t,)))
            ops.append(Op("RZ", (), (t,), -1, math.pi / float(1 << k)))
        ops.append(Op("RZ", (), (t,), -1, math.pi / float(1 << (k + 1))))
    return ops, n


def haar(k: int, rng: np.random.Generator) -> np.ndarray:
    d = 1 << k
    z = rng.standard_normal((d, d)) + 1j * rng.standard_normal((d, d))
    q, r = np.linalg.qr(z / math.sqrt(2.0))
    ph = np.diag(r) / np.abs(np.diag(r))
    return (q * ph[None, :]).astype(np.complex128)


MIX = ("H", "X", "RX", "RY", "RZ", "RY", "T", "S", "CX", "CX", "CX", "CZ", "CP", "CRY", "SWAP", "U2", "U4", "CCX")


def mixed(n: int, depth: int, structure: int, seed: int) -> Tuple[List[Op], int]:
    """Gates of every kind on random qubits; the structure is fixed by ``structure``, matrices come from the seed."""
    place, values = random.Random(structure), np.random.default_rng(seed)
    ops: List[Op] = [Op("H", (), (q,)) for q in range(n)]
    npar = 0
    for _ in range(depth * n):
        g = place.choice(MIX)
        q = tuple(place.sample(range(n), 3))
        if g in ("RX", "RY", "RZ"):
            ops.append(Op(g, (), q[:1], npar))
            npar += 1
        elif g in ("CP", "CRY"):
            ops.append(Op("PHASE" if g == "CP" else "RY", q[:1], q[1:2], npar))
            npar += 1
        elif g in ("CX", "CZ"):
            ops.append(Op(g[1], q[:1], q[1:2]))
        elif g == "CCX":
            ops.append(Op("X", q[:2], q[2:]))
        elif g == "SWAP":
            ops.append(Op("SWAP", (), q[:2]))
        elif g in ("U2", "U4"):
            k = 1 if g == "U2" else 2
            ops.append(Op(g, (), q[:k], -1, 0.0, haar(k, values)))
        else:
            ops.append(Op(g, (), q[:1]))
    return ops, npar


def circuit_of(case: dict, seed: int) -> Tuple[List[Op], int]:
    if case["circuit"] == "hea":
        return hea(case["n"], case["layers"])
    if case["circuit"] == "qft":
        return qft(case["n"])
    if case["circuit"] == "universal":
        return universal(case["n"])
    return mixed(case["n"], case["layers"], case["structure"], seed)


def batch_sizes(case: dict) -> List[Tuple[int, int]]:
    """(qubits, layers) of each circuit of a batch."""
    r = random.Random(case["structure"])
    return [(r.randint(case["qmin"], case["qmax"]), r.randint(case["lmin"], case["lmax"])) for _ in range(case["count"])]


def angles(count: int, seed: int) -> np.ndarray:
    return np.random.default_rng(seed).uniform(0.0, 2.0 * math.pi, size=count)


def gate_list(case: dict, seed: int) -> List[Op]:
    """One gate of every class on low, middle and high qubits: the targets and controls of the single-gate sweep."""
    n = case["n"]
    r, values = random.Random(case["structure"]), np.random.default_rng(seed)
    ops: List[Op] = []
    for g in ("X", "H", "RZ", "RY", "U2", "Z", "CX", "SWAP", "U4", "CCX", "CP"):
        for region in (0, 1, 2):
            lo, hi = region * n // 3, (region + 1) * n // 3
            t = r.randrange(lo, hi)
            c = r.choice([q for q in (0, n // 2, n - 1) if q != t])
            d = r.choice([q for q in range(n) if q not in (t, c)])
            th = float(values.uniform(0, 2 * math.pi))
            if g == "U2":
                ops.append(Op("U2", (), (t,), -1, 0.0, haar(1, values)))
            elif g == "U4":
                ops.append(Op("U4", (), (c, t), -1, 0.0, haar(2, values)))
            elif g == "CX":
                ops.append(Op("X", (c,), (t,)))
            elif g == "CCX":
                ops.append(Op("X", (c, d), (t,)))
            elif g == "CP":
                ops.append(Op("PHASE", (c,), (t,), -1, th))
            elif g == "SWAP":
                ops.append(Op("SWAP", (), (c, t)))
            else:
                ops.append(Op(g, (), (t,), -1, th if g in ("RZ", "RY") else 0.0))
    return ops


def chain_terms(n: int, kind: str) -> List[Tuple[float, str, Tuple[int, ...]]]:
    """Heisenberg chain with a field, or the transverse-field Ising chain."""
    terms: List[Tuple[float, str, Tuple[int, ...]]] = []
    for q in range(n - 1):
        if kind == "heisenberg":
            terms += [(0.5, "XX", (q, q + 1)), (0.5, "YY", (q, q + 1))]
        terms.append((1.0 if kind == "ising" else 0.75, "ZZ", (q, q + 1)))
    for q in range(n):
        terms.append((0.9, "X", (q,)) if kind == "ising" else (0.25, "Z", (q,)))
    return terms


def dense_list(case: dict, seed: int) -> List[Tuple[Tuple[int, ...], np.ndarray]]:
    """Blocks of 4 to 6 qubits on the lowest, the highest and scattered qubits."""
    n = case["n"]
    r, values = random.Random(case["structure"]), np.random.default_rng(seed)
    out = []
    for k in (4, 5, 6):
        for qs in (tuple(range(k)), tuple(range(n - k, n)), tuple(r.sample(range(n), k))):
            out.append((qs, haar(k, values)))
    return out


# --------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------
def listed() -> List[dict]:
    return [
        # a step of a small variational optimisation: launches and host work count
        dict(name="train_12q_c128", kind="train", n=12, layers=4, circuit="hea", dtype="c128", obs="sum_zz"),
        # the 24-qubit gradient the library is benchmarked on
        dict(name="train_24q_c128", kind="train", n=24, layers=8, circuit="hea", dtype="c128", obs="sum_zz"),
        # an ensemble of circuits of mixed sizes, single precision
        dict(name="batch_48_c64", kind="batch", count=48, qmin=14, qmax=20, lmin=4, lmax=12, structure=1006,
             dtype="c64", obs="sum_zz"),
        # large circuits run once: ansatz, Fourier transform, universal circuit, and arbitrary gates
        dict(name="hea_29q_c128", kind="forward", n=29, layers=10, circuit="hea", dtype="c128", obs="sum_z"),
        dict(name="qft_30q_c64", kind="forward", n=30, layers=1, circuit="qft", dtype="c64", obs="sum_z"),
        dict(name="universal_28q_c128", kind="forward", n=28, layers=1, circuit="universal", dtype="c128", obs="sum_z"),
        dict(name="mixed_27q_c64", kind="forward", n=27, layers=8, circuit="mixed", structure=11, dtype="c64",
             obs="sum_zz"),
        # gates applied call by call to the 16 GiB state of the gate benchmark
        dict(name="gates_30q_c128", kind="gates", n=30, structure=3, dtype="c128"),
        # a small circuit applied op by op and measured: one launch per gate
        dict(name="ops_13q_c64", kind="ops", n=13, layers=4, circuit="mixed", structure=5, dtype="c64", mode="plain",
             ham="ising"),
        # the gradient of a Hamiltonian the fused engine does not take
        dict(name="adjoint_21q_c128", kind="adjoint", n=21, layers=4, circuit="hea", dtype="c128", ham="ising"),
        # measuring a Heisenberg chain
        dict(name="pauli_27q_c128", kind="pauli", n=27, dtype="c128", ham="heisenberg"),
        # dense blocks on the matrix cores
        dict(name="dense_27q_c64", kind="dense", n=27, structure=7, dtype="c64"),
    ]


def draw(rng: random.Random) -> dict:
    kind = rng.choice(("train", "train", "batch", "forward", "forward", "forward", "gates", "ops", "ops", "adjoint",
                       "pauli", "dense"))
    dtype = rng.choice(("c128", "c64"))
    obs = rng.choice(("sum_z", "sum_zz"))
    ham = rng.choice(("ising", "heisenberg"))
    structure = rng.randrange(1 << 20)
    if kind == "train":
        return dict(kind=kind, n=rng.randint(8, 24), layers=rng.randint(2, 8), circuit="hea", dtype=dtype, obs=obs)
    if kind == "batch":
        qmin = rng.randint(8, 16)
        lmin = rng.randint(2, 6)
        return dict(kind=kind, count=rng.randint(4, 48), qmin=qmin, qmax=rng.randint(qmin, 20), lmin=lmin,
                    lmax=rng.randint(lmin, 12), structure=structure, dtype=dtype, obs=obs)
    if kind == "forward":
        circuit = rng.choice(("hea", "qft", "universal", "mixed"))
        n = rng.randint(14, {"hea": 28, "qft": 29, "universal": 28, "mixed": 26}[circuit])
        return dict(kind=kind, n=n, layers=rng.randint(2, 10), circuit=circuit, structure=structure, dtype=dtype,
                    obs=obs)
    if kind == "gates":
        return dict(kind=kind, n=rng.randint(16, 29), structure=structure, dtype=dtype)
    if kind == "ops":
        circuit = rng.choice(("hea", "qft", "mixed"))
        return dict(kind=kind, n=rng.randint(8, 24), layers=rng.randint(2, 4), circuit=circuit, structure=structure,
                    dtype=dtype, mode=rng.choice(("plain", "fused", "blocks")), ham=ham)
    if kind == "adjoint":
        return dict(kind=kind, n=rng.randint(8, 21), layers=rng.randint(2, 4), circuit="hea", dtype=dtype, ham=ham)
    if kind == "pauli":
        return dict(kind=kind, n=rng.randint(12, 27), dtype=dtype, ham=ham)
    return dict(kind="dense", n=rng.randint(14, 27), structure=structure, dtype=dtype)


def gaussian(n: int, dtype: str, seed: int) -> torch.Tensor:
    """A normalised Gaussian state on the GPU."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    v = torch.randn(1 << n, dtype=TORCH[dtype], device="cuda", generator=g)
    return v.div_(torch.linalg.vector_norm(v))


def prepare(case: dict, seed: int) -> Dict[str, object]:
    kind, dtype = case["kind"], case["dtype"]
    s: Dict[str, object] = {"kind": kind, "case": case}
    if kind in ("train", "forward"):
        ops, npar = circuit_of(case, seed)
        s["batch"] = sv.Batch([(case["n"], ops, npar, case["obs"])], dtype=dtype, with_grad=kind == "train")
        s["params"] = torch.from_numpy(angles(npar, seed)).cuda()
        if kind == "train":
            s["params"].requires_grad_(True)
        else:
            s["e"] = torch.zeros(1, dtype=torch.float64, device="cuda")
            s["g"] = torch.zeros(1, dtype=torch.float64, device="cuda")
    elif kind == "batch":
        circuits, npar = [], 0
        for n, layers in batch_sizes(case):
            ops, k = hea(n, layers)
            circuits.append((n, ops, k, case["obs"]))
            npar += k
        s["batch"] = sv.Batch(circuits, dtype=dtype, with_grad=True)
        s["params"] = torch.from_numpy(angles(npar, seed)).cuda()
        s["e"] = torch.zeros(len(circuits), dtype=torch.float64, device="cuda")
        s["g"] = torch.zeros(npar, dtype=torch.float64, device="cuda")
    elif kind == "gates":
        s["psi"] = sv.State(case["n"], dtype, tensor=gaussian(case["n"], dtype, seed), basis=None)
        s["ops"] = gate_list(case, seed)
    elif kind == "ops":
        ops, npar = circuit_of(case, seed)
        s["psi"] = sv.State(case["n"], dtype)
        s["circuit"] = sv.Circuit(case["n"], ops, npar)
        s["params"] = angles(npar, seed)
        s["ham"] = sv.Observable(chain_terms(case["n"], case["ham"]))
    elif kind == "adjoint":
        ops, npar = circuit_of(case, seed)
        s["psi"], s["lam"] = sv.State(case["n"], dtype), sv.State(case["n"], dtype)
        s["circuit"] = sv.Circuit(case["n"], ops, npar)
        s["params"] = torch.from_numpy(angles(npar, seed)).requires_grad_(True)
        s["ham"] = sv.Observable(chain_terms(case["n"], case["ham"]))
    elif kind == "pauli":
        s["psi"] = sv.State(case["n"], dtype, tensor=gaussian(case["n"], dtype, seed), basis=None)
        s["ham"] = sv.Observable(chain_terms(case["n"], case["ham"]))
    else:
        s["psi"] = sv.State(case["n"], dtype, tensor=gaussian(case["n"], dtype, seed), basis=None)
        s["blocks"] = dense_list(case, seed)
    return s


def run(s: Dict[str, object]):
    kind = s["kind"]
    if kind == "train":
        p = s["params"]
        p.grad = None
        e = sv.AdjointExpval.apply(p, s["batch"])
        e.backward()
        return {"e": e.detach(), "grad": p.grad}
    if kind == "batch":
        s["batch"].run_device(s["params"], s["e"], s["g"])
        return {"e": s["e"], "grad": s["g"]}
    if kind == "forward":
        s["batch"].run_device(s["params"], s["e"], s["g"])
        psi = s["batch"].state_tensor(0)
        psi.owner = s["batch"]  # the view is valid while its batch lives
        return {"e": s["e"], "psi": psi}
    if kind == "gates":
        psi = s["psi"]
        for o in s["ops"]:
            psi.apply(o.gate, o.targets, o.controls, (o.value,), o.matrix)
        return {"psi": psi.tensor}
    if kind == "ops":
        psi, mode = s["psi"].set_basis(0), s["case"]["mode"]
        s["circuit"].apply(psi, s["params"], fuse_diagonal=mode == "fused", dense_block=5 if mode == "blocks" else 0)
        return {"e": psi.expval(s["ham"]), "psi": psi.tensor}
    if kind == "adjoint":
        p = s["params"]
        p.grad = None
        e = sv.AdjointExpval.apply(p, s["circuit"], s["psi"], s["lam"], s["ham"])
        e.backward()
        return {"e": e.detach(), "grad": p.grad}
    if kind == "pauli":
        return {"e": s["psi"].expval(s["ham"]), "norm2": s["psi"].norm2()}
    for qs, m in s["blocks"]:
        s["psi"].apply_dense(qs, m)
    return {"psi": s["psi"].tensor}


# --------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------
def gate_flops(o: Op) -> float:
    """Operations per amplitude of the state (a controlled gate touches its share)."""
    share = 0.5 ** len(o.controls)
    if o.gate in ("X", "SWAP", "I"):
        return 0.0
    if o.gate in ("Z", "S", "T", "PHASE"):
        return 3.0 * share
    if o.gate in ("RZ", "RY", "H"):
        return 6.0 * share
    return (30.0 if o.gate == "U4" else 14.0) * share


def gate_bytes(o: Op) -> float:
    """Share of the state read and written."""
    share = 0.5 ** len(o.controls)
    return share * (0.5 if o.gate in ("Z", "S", "T", "PHASE", "SWAP") else 1.0)


def work(case: dict) -> Dict[str, float]:
    kind, size = case["kind"], SIZE[case["dtype"]]
    if kind == "batch":
        flops = bytes_ = 0.0
        for n, layers in batch_sizes(case):
            ops, npar = hea(n, layers)
            flops += (1 << n) * (3.0 * sum(gate_flops(o) for o in ops) + 4.0 * npar)
            bytes_ += 16.0 * npar
        return {"bytes": bytes_ + 8.0 * case["count"], "flops": flops}
    n = case["n"]
    amps = float(1 << n)
    if kind == "gates":
        ops = gate_list(case, 0)
        return {"bytes": 2.0 * size * amps * sum(gate_bytes(o) for o in ops),
                "flops": amps * sum(gate_flops(o) for o in ops)}
    if kind == "pauli":
        return {"bytes": 2.0 * size * amps, "flops": amps * (4.0 + 4.0 * len(chain_terms(n, case["ham"])))}
    if kind == "dense":
        return {"bytes": 2.0 * size * amps * len(dense_list(case, 0)), "flops": amps * 3.0 * (8 * 16 + 8 * 32 + 8 * 64)}
    ops, npar = circuit_of(case, 0)
    flops = amps * sum(gate_flops(o) for o in ops)
    if kind in ("train", "adjoint"):
        return {"bytes": 16.0 * npar + 8.0, "flops": 3.0 * flops + 4.0 * amps * npar}
    return {"bytes": size * amps + 8.0 * npar, "flops": flops}


# --------------------------------------------------------------------------
# the same outputs from plain torch in complex128
# --------------------------------------------------------------------------
def part(v: torch.Tensor, n: int, bits: Dict[int, int]) -> torch.Tensor:
    """View of the amplitudes whose bit q is bits[q] for every q."""
    shape, index, top = [], [], n
    for q in sorted(bits, reverse=True):
        shape += [1 << (top - q - 1), 2]
        index += [slice(None), bits[q]]
        top = q
    return v.view(shape + [1 << top])[tuple(index) + (slice(None),)]


def matrix_of(o: Op, params: np.ndarray) -> np.ndarray:
    th = params[o.pidx] if o.pidx >= 0 else o.value
    c, s = math.cos(th / 2), math.sin(th / 2)
    r = math.sqrt(0.5)
    if o.matrix is not None:
        return o.matrix
    return np.array({
        "X": [[0, 1], [1, 0]], "H": [[r, r], [r, -r]], "Z": [[1, 0], [0, -1]], "S": [[1, 0], [0, 1j]],
        "T": [[1, 0], [0, complex(r, r)]], "RX": [[c, -1j * s], [-1j * s, c]], "RY": [[c, -s], [s, c]],
        "RZ": [[complex(c, -s), 0], [0, complex(c, s)]], "PHASE": [[1, 0], [0, complex(math.cos(th), math.sin(th))]],
        "SWAP": [[1, 0, 0, 0], [0, 0, 1, 0], [0, 1, 0, 0], [0, 0, 0, 1]],
    }[o.gate], dtype=np.complex128)


def apply_matrix(v: torch.Tensor, n: int, controls, targets, m: np.ndarray) -> None:
    """v <- m on targets (the first-listed is the most significant bit), where every control is 1; in place."""
    k = len(targets)
    sides = []
    for a in range(1 << k):
        bits = {c: 1 for c in controls}
        bits.update({t: (a >> (k - 1 - j)) & 1 for j, t in enumerate(targets)})
        sides.append(part(v, n, bits))
    rows = [a for a in range(1 << k) if any(m[a, b] != (1 if a == b else 0) for b in range(1 << k))]
    if not np.any(m - np.diag(np.diag(m))):
        for a in rows:
            sides[a].mul_(complex(m[a, a]))
        return
    old = [x.clone() for x in sides]
    for a in rows:
        sides[a].mul_(complex(m[a, a]))
        for b in range(1 << k):
            if b != a and m[a, b] != 0:
                sides[a].add_(old[b], alpha=complex(m[a, b]))


def zero_state(n: int) -> torch.Tensor:
    v = torch.zeros(1 << n, dtype=torch.complex128, device="cuda")
    v[0] = 1.0
    return v


def forward_exact(n: int, ops: List[Op], params: np.ndarray) -> torch.Tensor:
    v = zero_state(n)
    for o in ops:
        apply_matrix(v, n, o.controls, o.targets, matrix_of(o, params))
    return v


def pauli_applied(v: torch.Tensor, n: int, letters: str, qubits) -> torch.Tensor:
    w = v.clone()
    p = {"X": np.array([[0, 1], [1, 0]]), "Y": np.array([[0, -1j], [1j, 0]]), "Z": np.diag([1, -1])}
    for c, q in zip(letters, qubits):
        apply_matrix(w, n, (), (q,), p[c].astype(np.complex128))
    return w


def energy(v: torch.Tensor, n: int, terms) -> Tuple[float, torch.Tensor]:
    """<v|O|v> and O v."""
    out = torch.zeros_like(v)
    for c, letters, qubits in terms:
        out.add_(pauli_applied(v, n, letters, qubits), alpha=c)
    return float(torch.view_as_real(v).mul(torch.view_as_real(out)).sum()), out


def plain_terms(obs: str, n: int):
    if obs == "sum_z":
        return [(1.0, "Z", (q,)) for q in range(n)]
    return [(1.0, "ZZ", (q, q + 1)) for q in range(n - 1)]


def gradient_exact(n: int, ops: List[Op], npar: int, params: np.ndarray, terms) -> Tuple[float, np.ndarray]:
    """Energy and its derivatives: dE = Im<lambda|G|phi> for exp(-i theta G / 2), walked backwards."""
    phi = forward_exact(n, ops, params)
    e, lam = energy(phi, n, terms)
    g = [torch.zeros((), dtype=torch.float64, device="cuda")] * npar
    for o in reversed(ops):
        if o.pidx >= 0:
            a, b = part(phi, n, {o.targets[0]: 0}), part(phi, n, {o.targets[0]: 1})
            x, y = part(lam, n, {o.targets[0]: 0}), part(lam, n, {o.targets[0]: 1})
            if o.gate == "RY":  # G = Y
                d = (x.conj() * b).mul_(-1j).sum() + (y.conj() * a).mul_(1j).sum()
            else:  # RZ: G = Z
                d = (x.conj() * a).sum() - (y.conj() * b).sum()
            g[o.pidx] = g[o.pidx] + d.imag
        m = matrix_of(o, params).conj().T
        apply_matrix(phi, n, o.controls, o.targets, m)
        apply_matrix(lam, n, o.controls, o.targets, m)
    return e, torch.stack(g).cpu().numpy()


def apply_dense_exact(v: torch.Tensor, n: int, qubits, m: np.ndarray) -> torch.Tensor:
    """The block as one matrix product over the state with the block's qubits moved to the front."""
    order = sorted(qubits, reverse=True)
    shape, axis, top = [], {}, n
    for q in order:
        shape += [1 << (top - q - 1), 2]
        axis[q] = len(shape) - 1
        top = q
    shape.append(1 << top)
    front = [axis[q] for q in qubits]
    perm = front + [d for d in range(len(shape)) if d not in front]
    x = v.view(shape).permute(perm).contiguous()
    y = torch.mm(torch.from_numpy(m).cuda(), x.view(1 << len(qubits), -1)).view(x.shape)
    back = [perm.index(d) for d in range(len(shape))]
    return y.permute(back).contiguous().view(-1)


def exact(case: dict, seed: int):
    kind = case["kind"]
    if kind == "batch":
        sizes = batch_sizes(case)
        if sum(3 * n * layers for n, layers in sizes) > 40000:
            return None
        params, at, es, gs = angles(sum(2 * n * layers for n, layers in sizes), seed), 0, [], []
        for n, layers in sizes:
            ops, npar = hea(n, layers)
            e, g = gradient_exact(n, ops, npar, params[at:at + npar], plain_terms(case["obs"], n))
            at += npar
            es.append(e)
            gs.append(g)
        return {"e": np.array(es), "grad": np.concatenate(gs)}
    n = case["n"]
    if kind == "gates":
        v = gaussian(n, case["dtype"], seed).to(torch.complex128)
        for o in gate_list(case, seed):
            apply_matrix(v, n, o.controls, o.targets, matrix_of(o, np.zeros(0)))
        return {"psi": v}
    if kind == "dense":
        v = gaussian(n, case["dtype"], seed).to(torch.complex128)
        for qs, m in dense_list(case, seed):
            v = apply_dense_exact(v, n, qs, m)
        return {"psi": v}
    if kind == "pauli":
        v = gaussian(n, case["dtype"], seed).to(torch.complex128)
        return {"e": energy(v, n, chain_terms(n, case["ham"]))[0], "norm2": float(torch.view_as_real(v).square().sum())}
    ops, npar = circuit_of(case, seed)
    params = angles(npar, seed)
    if kind in ("train", "adjoint"):
        terms = plain_terms(case["obs"], n) if kind == "train" else chain_terms(n, case["ham"])
        e, g = gradient_exact(n, ops, npar, params, terms)
        return {"e": np.array(e), "grad": g}
    v = forward_exact(n, ops, params)
    if kind == "ops":
        return {"e": energy(v, n, chain_terms(n, case["ham"]))[0], "psi": v}
    e = 0.0
    for _, _, qubits in plain_terms(case["obs"], n):
        if len(qubits) == 1:
            e += sum((1 - 2 * a) * weight(v, n, {qubits[0]: a}) for a in (0, 1))
        else:
            e += sum((1 - 2 * (a ^ b)) * weight(v, n, {qubits[0]: a, qubits[1]: b}) for a in (0, 1) for b in (0, 1))
    return {"e": np.array([e]), "psi": v}


def weight(v: torch.Tensor, n: int, bits: Dict[int, int]) -> float:
    """Probability of reading bits."""
    x = part(v, n, bits)
    return float(x.real.square().sum() + x.imag.square().sum())
