"""sv_circuit_apply on small states in complex64: the same bits as gate by gate.

One kernel runs the whole circuit on states of at most 2^14 amplitudes (with few gates besides 4x4 ones, single-gate
launches do at 2^14); it rounds every product as the single-gate kernels do, so the amplitudes are the same bits.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

sv = pytest.importorskip("paper_2508_13615_amd")
Op = W.Op
KINDS = ("I", "X", "Y", "Z", "H", "S", "T", "RX", "RY", "RZ", "PHASE", "U2", "SWAP", "U4")


def circuit(n, kinds, count, seed):
    rng = np.random.default_rng(seed)
    ops = []
    for i in range(count):
        g = kinds[i % len(kinds)]
        nt = 2 if g in ("SWAP", "U4") else 1
        q = [int(x) for x in rng.permutation(n)]
        nc = int(rng.integers(0, min(3, n - nt) + 1)) if g != "U4" else int(rng.integers(0, min(2, n - nt) + 1))
        m = W.haar_unitary(nt, rng) if g in ("U2", "U4") else None
        ops.append(Op(g, tuple(q[nt:nt + nc]), tuple(q[:nt]), -1, float(rng.uniform(-6, 6)), m))
    return ops


def check(n, ops, seed):
    psi0 = W.gaussian_state(n, seed).astype(np.complex64)
    one = sv.State(n, "c64").load(psi0)
    for o in ops:
        one.apply(o.gate, o.targets, o.controls, [o.value], o.matrix)
    st = sv.State(n, "c64").load(psi0)
    sv.Circuit(n, ops).apply(st)
    assert np.array_equal(st.numpy().view(np.float32), one.numpy().view(np.float32))


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n", [2, 4, 7, 12, 13, 14])
def test_each_gate_kind(n, kind):
    check(n, circuit(n, (kind,), 10, n), 30 + n)


@pytest.mark.parametrize("n", [13, 14, 15])
@pytest.mark.parametrize("kinds", [("U4",), ("U4", "U4", "H"), ("H", "U4"), KINDS])
@pytest.mark.parametrize("count", [2, 3, 5, 6, 60])
def test_around_the_rule_at_the_largest_states(n, kinds, count):
    check(n, circuit(n, kinds, count, count), 40 + n)
