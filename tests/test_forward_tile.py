"""Forward-only complex128 runs of large circuits take a larger tile where that saves passes.

The rule on the host (fewer passes than the tuned 2^10 tile from 24 qubits up, the same plan below and with gradients),
and the state and energy of the larger tile against the tuned one.  Both apply the same gates in double: each
amplitude vector is off by at most a few eps a gate, the energy by that times the n terms of the observable.
"""
import numpy as np
import pytest

import workloads as W

sv = pytest.importorskip("paper_2508_13615_amd")
Op = W.Op


def layers(n, depth):
    """Rotations, then a ring of CX, on every qubit: few ops a pass."""
    ops, k = [], 0
    for _ in range(depth):
        for q in range(n):
            ops += [Op("RY", (), (q,), k), Op("RZ", (), (q,), k + 1)]
            k += 2
        ops += [Op("X", (q,), ((q + 1) % n,)) for q in range(n)]
    return ops, k


def every_form(n, depth):
    """All kinds that reach the rule: controlled gates, phases, swaps, dense and diagonal 2x2, far and near qubits."""
    rng = np.random.default_rng(n)
    ops, k = [Op("H", (), (q,)) for q in range(n)], 0
    for _ in range(depth):
        for q in range(n):
            a, b = (int(x) for x in rng.choice([x for x in range(n) if x != q], size=2, replace=False))
            ops += [Op("RX", (), (q,), k), Op("PHASE", (a,), (q,), k), Op("U2", (), (b,), -1, 0.0, W.haar_unitary(1, rng))]
            ops += [Op("SWAP", (), (q, a))] if q % 5 == 0 else [Op("X", (a, b), (q,))] if q % 7 == 0 else []
            k += 1
        ops += [Op("RZ", (q,), (n - 1 - q,), q) for q in range(n // 2)]
    return ops, k


def test_rule():
    def passes(n, **kw):
        ops, k = layers(n, 4)
        return sv.batch_plan([(n, ops, k, "sum_z")], **kw)["passes"]

    assert passes(24, with_grad=False) < passes(24, with_grad=False, tile_qubits=10)
    assert passes(23, with_grad=False) == passes(23, with_grad=False, tile_qubits=10)
    assert passes(24) == passes(24, tile_qubits=10)


@pytest.mark.gpu
@pytest.mark.parametrize("n,form", [(24, layers), (25, layers), (24, every_form), (25, every_form)])
def test_larger_tile_same_state(n, form):
    ops, k = form(n, 3)
    theta = np.random.default_rng(n).uniform(-np.pi, np.pi, k)
    circuit = [(n, ops, k, "sum_zz")]
    a = sv.Batch(circuit, with_grad=False)
    b = sv.Batch(circuit, with_grad=False, tile_qubits=10)
    assert a.info()["passes"] <= b.info()["passes"] - (form is layers)
    ea, eb = (float(np.asarray(x.run(theta)[0]).ravel()[0]) for x in (a, b))
    bar = 8 * len(ops) * np.finfo(np.float64).eps
    assert float((a.state_tensor(0) - b.state_tensor(0)).abs().max()) <= bar
    assert abs(ea - eb) <= n * bar
