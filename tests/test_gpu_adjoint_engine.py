"""Circuit.adjoint_grad on complex128 states (the pass engine on the caller's states), against the fp64 oracle.

From a random state, not |0...0>: the energy and gradient of a general Pauli sum against the oracle's central
differences (1e-7), every gate kind and shared parameters, at sizes below, at and above a tile; psi holds its input
state again afterwards (1e-12); a second call with other parameters, and a circuit with a gate too wide for the
engine's tile, which takes the op-by-op sweep.
"""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu

sv = pytest.importorskip("paper_2508_13615_amd")
Op = W.Op


def circuit(n, seed):
    rng = np.random.default_rng(seed)
    ops, p = [], 0
    for k in range(4 * n):
        q = [int(x) for x in rng.permutation(n)[:3]]
        g = int(rng.integers(0, 9)) if n > 2 else int(rng.integers(0, 3))
        if g < 3:
            ops.append(Op(("RX", "RY", "RZ")[g], (), (q[0],), p % 7))
            p += 1
        elif g == 3:
            ops.append(Op("PHASE", (q[0],), (q[1],), p % 7))
            p += 1
        elif g == 4:
            ops.append(Op("RY", (q[0],), (q[1],), p % 7))
            p += 1
        elif g == 5:
            ops.append(Op("X", (q[0],), (q[1],)))
        elif g == 6:
            ops.append(Op("SWAP", (), (q[0], q[1])))
        elif g == 7:
            ops.append(Op("U4", (), (q[0], q[1]), -1, 0.0, W.haar_unitary(2, rng)))
        else:
            ops.append(Op("X", (q[0], q[1]), (q[2],)))
    return ops + [Op("RY", (), (0,), k) for k in range(7)]  # every parameter is used


def terms(n):
    t = [(0.7, "Z", (q,)) for q in range(n)] + [(0.4, "X", (q,)) for q in range(0, n, 2)]
    return t + ([(0.3, "YX", (0, n - 1)), (0.2, "ZZ", (0, 1))] if n > 1 else [])


@pytest.mark.parametrize("n", [1, 2, 3, 6, 10, 11, 12, 13])
def test_adjoint_from_a_random_state(n):
    psi0 = W.gaussian_state(n, 40 + n)
    ops = circuit(n, n)
    circ = sv.Circuit(n, ops, 7)
    psi, lam = sv.State(n), sv.State(n)
    for seed in (1, 2):
        th = W.uniform_angles(7, seed)
        e, g = circ.adjoint_grad(psi.load(psi0), lam, th, terms(n))
        assert abs(e - oracle.energy(n, ops, th, terms(n), init=psi0)) <= 1e-12 * len(terms(n))
        assert float(np.max(np.abs(psi.numpy() - psi0))) <= 1e-12
        h = 1e-6
        for k in range(7):
            up, dn = th.copy(), th.copy()
            up[k] += h
            dn[k] -= h
            fd = (oracle.energy(n, ops, up, terms(n), init=psi0) - oracle.energy(n, ops, dn, terms(n), init=psi0)) / (2 * h)
            assert abs(g[k] - fd) <= 1e-7, (k, g[k], fd)


def test_a_gate_wider_than_a_tile_walks_op_by_op():
    n = 12
    ops = [Op("H", (), (q,)) for q in range(n)] + [Op("RY", (), (q,), q) for q in range(n)]
    ops += [Op("SWAP", tuple(range(6)), (10, 11)), Op("RX", (3,), (7,), 4)]
    th = W.uniform_angles(n, 5)
    circ = sv.Circuit(n, ops, n)
    tuned = sv.tune_engine_get("c128", True)
    sv.tune_engine_set("c128", True, 6, 8)  # a tile of 6 qubits, the SWAP has 8
    try:
        e, g = circ.adjoint_grad(sv.State(n), sv.State(n), th, terms(n))
    finally:
        sv.tune_engine_set("c128", True, *tuned)
    assert abs(e - oracle.energy(n, ops, th, terms(n))) <= 1e-12 * len(terms(n))
    ref = oracle.fd_grad(n, ops, th, terms(n), which=[0, 4, 11])
    assert float(np.max(np.abs((g - ref)[[0, 4, 11]]))) <= 1e-7
