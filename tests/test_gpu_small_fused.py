"""Circuit.apply(fuse_diagonal=True) on states that fit one workgroup.

The call sums a diagonal run's phases as angles and applies the sum once, so a run whose angles add up to quarter
turns moves amplitudes exactly, in both dtypes: no rounding per gate, on these sizes as on larger ones.
"""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu

sv = pytest.importorskip("paper_2508_13615_amd")
Op = W.Op


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n", [1, 2, 6, 12, 13, 14, 15])
def test_runs_of_quarter_turns_are_exact(n, dtype):
    q = n // 2
    ops = [Op("T", (), (q,)), Op("T", (), (q,)), Op("S", (), (q,)), Op("Z", (), (q,))]  # 1/8 + 1/8 + 1/4 + 1/2 turns
    ops += [Op("T", (), (0,)) for _ in range(10)]  # 10/8 turns: S
    psi0 = W.gaussian_state(n, 70 + n).astype(np.complex128 if dtype == "c128" else np.complex64)
    st = sv.State(n, dtype).load(psi0)
    sv.Circuit(n, ops).apply(st, fuse_diagonal=True)
    ref = psi0.copy()
    one = (np.arange(1 << n) & 1) == 1
    ref.real[one], ref.imag[one] = -psi0.imag[one], psi0.real[one]
    assert np.array_equal(st.numpy(), ref)


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n", [2, 5, 11, 13])
def test_quarter_turns_on_several_masks_are_exact(n, dtype):
    """S, Z and their controlled forms on up to eight masks: every amplitude's angle is a sum of quarter turns."""
    rng = np.random.default_rng(n)
    for count in (2, 3, 4, 5, 9, 24):
        ops, turns, x = [Op("SWAP", (), (0, 1))], np.zeros(1 << n, dtype=int), np.arange(1 << n)
        for _ in range(count):
            q = [int(v) for v in rng.permutation(n)[:int(rng.integers(1, min(n, 3) + 1))]]
            g = str(rng.choice(["S", "Z"]))
            ops.append(Op(g, tuple(q[1:]), (q[0],)))
            turns += (1 if g == "S" else 2) * np.logical_and.reduce([(x >> v) & 1 for v in q])
        psi0 = W.gaussian_state(n, 30 + n).astype(np.complex128 if dtype == "c128" else np.complex64)
        st = sv.State(n, dtype).load(psi0)
        sv.Circuit(n, ops).apply(st, fuse_diagonal=True)
        ref = psi0[(x & ~3) | ((x & 1) << 1) | ((x >> 1) & 1)]
        for k in range(1, 4):
            at, z = turns % 4 == k, ref.copy()
            ref.real[at] = {1: -z.imag, 2: -z.real, 3: z.imag}[k][at]
            ref.imag[at] = {1: z.real, 2: -z.imag, 3: -z.real}[k][at]
        assert np.array_equal(st.numpy(), ref), count


@pytest.mark.parametrize("dtype,unit", [("c128", 2.0 ** -53), ("c64", 2.0 ** -24)])
@pytest.mark.parametrize("n", [2, 3, 7, 10, 11, 12, 13, 14])
@pytest.mark.parametrize("count", [2, 3, 4, 5, 8])
def test_a_run_rounds_once(n, dtype, unit, count):
    """A move and one run of controlled phases and RZs: relative to each amplitude, the phase's rounding and the
    product's (8 units); in complex128 also the angles' (sums of at most 8 angles up to 2 turns, times pi) and the
    oracle's own gate by gate (256 units in all).  In complex64 the larger states' launched form sums in float."""
    rng = np.random.default_rng(100 * n + count)
    ops = [Op("SWAP", (), (0, 1))]
    for i in range(count):
        q = [int(v) for v in rng.permutation(n)[:2]]
        ops.append(Op("RZ", (), (q[0],), -1, float(rng.uniform(-6, 6))) if i % 3 == 1 else Op("PHASE", (q[0],), (q[1],), -1, float(rng.uniform(-6, 6))))
    psi0 = W.gaussian_state(n, 20 + n).astype(np.complex128 if dtype == "c128" else np.complex64)
    st = sv.State(n, dtype).load(psi0)
    sv.Circuit(n, ops).apply(st, fuse_diagonal=True)
    ref = oracle.run_circuit(psi0.astype(np.complex128), ops)
    bound = 256 if dtype == "c128" or n > 10 else 8
    assert float(np.max(np.abs(st.numpy() - ref) / np.abs(ref))) <= bound * unit


@pytest.mark.parametrize("dtype,tol", [("c128", 1e-12), ("c64", 1e-5)])
@pytest.mark.parametrize("n", [4, 9, 12, 13, 14])
def test_circuits_of_every_grouping(n, dtype, tol):
    """Composed gates, gates before runs of 1 to 70 terms, runs alone, moves and 4x4 gates between, across launches."""
    rng = np.random.default_rng(n)
    for size in (2, 6, 30):
        ops = []
        for _ in range(size):
            q = [int(v) for v in rng.permutation(n)]
            kind = int(rng.integers(6))
            if kind < 3:
                for g in rng.choice(["H", "RX", "RY", "X", "Y", "U2"], size=int(rng.integers(1, 4))):
                    ops.append(Op(str(g), (), (q[0],), -1, float(rng.uniform(-6, 6)), W.haar_unitary(1, rng) if g == "U2" else None))
            if kind > 0:
                for _ in range(int(rng.choice([1, 2, 3, 5, 12, 70], p=[.3, .2, .2, .15, .1, .05]))):
                    p = [int(v) for v in rng.permutation(n)]
                    g = str(rng.choice(["Z", "S", "T", "RZ", "PHASE", "I"]))
                    ops.append(Op(g, tuple(p[1:1 + int(rng.integers(0, 3))]), (p[0],), -1, float(rng.uniform(-6, 6))))
            if kind == 4:
                ops.append(Op("U4", (), (q[0], q[1]), -1, 0.0, W.haar_unitary(2, rng)))
            if kind == 5:
                ops.append(Op("SWAP", (q[2],), (q[0], q[1])))
        psi0 = W.gaussian_state(n, 60 + n).astype(np.complex128 if dtype == "c128" else np.complex64)
        st = sv.State(n, dtype).load(psi0)
        sv.Circuit(n, ops).apply(st, fuse_diagonal=True)
        ref = oracle.run_circuit(psi0.astype(np.complex128), ops)
        assert float(np.max(np.abs(st.numpy() - ref))) <= tol
