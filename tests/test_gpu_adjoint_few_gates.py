"""Circuit.adjoint_grad of circuits of one to three gates, on both sides of the rule that picks op by op or the engine.

One RY on qubit q of a basis state and sum_i Z_i: E = c0 + cos(theta) with gradient -sin(theta); more gates on other
qubits add to it.  Identity gates do not count.  Bars: 1e-12 per gate.
"""
import math

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

sv = pytest.importorskip("paper_2508_13615_amd")
Op = W.Op


@pytest.mark.parametrize("n", [3, 12, 20, 21, 23, 24])
@pytest.mark.parametrize("gates", [0, 1, 2, 3])
@pytest.mark.parametrize("off_diagonal", [False, True])
def test_few_gates(n, gates, off_diagonal):
    qs = (n - 1, 0, n // 2)[:gates]
    ops = [Op("I", (), (0,))] + [Op("RY", (), (q,), k) for k, q in enumerate(qs)] + [Op("I", (), (1,))]
    th = np.array([0.3, 1.1, 2.5])[:gates]
    obs = W.sum_z(n) + ([(0.5, "X", (n - 1,))] if off_diagonal else [])
    psi, lam = sv.State(n), sv.State(n)
    e, g = sv.Circuit(n, ops, gates).adjoint_grad(psi, lam, th, obs)
    ref_e = n - gates + float(np.sum(np.cos(th)))
    ref_g = -np.sin(th)
    if off_diagonal and gates:
        ref_e += 0.5 * math.sin(th[0])
        ref_g[0] += 0.5 * math.cos(th[0])
    assert abs(e - ref_e) <= 1e-12 * n
    assert gates == 0 or float(np.max(np.abs(g - ref_g))) <= 1e-12 * n
    assert abs(psi.expval([(1.0, "Z", (q,)) for q in range(n)]) - n) <= 1e-12 * n  # psi is |0...0> again
