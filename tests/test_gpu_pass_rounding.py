"""Which product a controlled 2x2 rounds first in complex64 passes: it decides the last bit of every amplitude.

Imaginary parts are fma(p, q, fl(r s)): with the control on a lane bit the product rounded by itself is Re u * Im z, on
a register bit Im u * Re z; real parts are fma(Re u, Re z, -fl(Im u * Im z)).  Energies and gradients of complex64 runs
are returned in double and show the difference, so the order is held here bit for bit: one controlled gate on a generic
state, recomputed from the state that the same run without the gate leaves.  The controls below lie on lane or register
bits in the layouts the planner makes for these circuits, and the gate runs last in them.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

sv = pytest.importorskip("paper_2508_13615_amd")
Op = W.Op
N = 10
LANE = {16: [(1, 4), (1, 5), (2, 6), (3, 4)], 8: [(1, 3), (2, 5), (1, 7), (2, 7)]}  # (target, control)
REG = {16: [(1, 8), (2, 9), (8, 9)], 8: [(1, 8), (2, 9), (8, 9)]}


def fma(a, b, c):
    return (a.astype(np.longdouble) * b.astype(np.longdouble) + c.astype(np.longdouble)).astype(np.float32)


def term(u, z, re_first):
    """u z as the kernel rounds it: (real part, imaginary part) before the sum over the two partners."""
    ur, ui = np.float32(u.real) * np.ones_like(z.real), np.float32(u.imag) * np.ones_like(z.real)
    x, y = z.real, z.imag
    return fma(ur, x, -(ui * y)), fma(ui, x, ur * y) if re_first else fma(ur, y, ui * x)


def run(ops, apt):
    b = sv.Batch([(N, ops, 0, "sum_z")], dtype="c64", tile_qubits=N, amps_per_thread=apt, with_grad=False)
    b.run([])
    return b.state(0)


@pytest.mark.parametrize("apt", [16, 8])
@pytest.mark.parametrize("where", ["lane", "register"])
def test_controlled_gate_rounds_in_its_order(apt, where):
    rng = np.random.default_rng(3)
    pre = [Op("U2", (), (q,), -1, 0.0, W.haar_unitary(1, rng)) for q in range(N)]
    pre += [Op("U4", (), (q, q + 1), -1, 0.0, W.haar_unitary(2, rng)) for q in range(0, N - 1, 2)]
    u = W.haar_unitary(1, rng)
    before = run(pre, apt)
    for t, c in (LANE if where == "lane" else REG)[apt]:
        after = run(pre + [Op("U2", (c,), (t,), -1, 0.0, u)], apt)
        x = np.arange(1 << N)
        lo = x[((x >> c) & 1 == 1) & ((x >> t) & 1 == 0)]
        hi = lo | (1 << t)
        ref = before.copy()
        for row, at in ((0, lo), (1, hi)):
            p, q = (term(u[row, k], before[z], where == "lane") for k, z in ((0, lo), (1, hi)))
            ref.real[at], ref.imag[at] = p[0] + q[0], p[1] + q[1]
        assert np.array_equal(after.view(np.float32), ref.view(np.float32)), (t, c)
