"""Circuits on states that fit one workgroup (k_small_circuit), against the fp64 oracle.

Every gate kind with zero to two controls from a random state, on the smallest states, at the largest the kernel takes
(128 KiB: 13 qubits complex128, 14 complex64) and one above, which goes gate by gate; more gates than one launch
holds, with 4x4 gates across its end; fused and plain application; moves bit-exact.  Bars as for single gates:
1e-12 (complex128), 1e-5 (complex64).
"""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu

sv = pytest.importorskip("paper_2508_13615_amd")
Op = W.Op
ONE = ("X", "Y", "Z", "H", "S", "T", "RX", "RY", "RZ", "PHASE", "U2", "I")


def circuit(n, count, seed):
    rng = np.random.default_rng(seed)
    ops = []
    for _ in range(count):
        q = [int(x) for x in rng.permutation(n)]
        g = str(rng.choice(ONE + ("SWAP", "U4", "U4"))) if n > 1 else str(rng.choice(ONE))
        nt = 2 if g in ("SWAP", "U4") else 1
        nc = int(rng.integers(0, min(2, n - nt) + 1)) if g != "U4" else int(rng.integers(0, min(1, n - nt) + 1))
        m = W.haar_unitary(nt, rng) if g in ("U2", "U4") else None
        ops.append(Op(g, tuple(q[nt:nt + nc]), tuple(q[:nt]), -1, float(rng.uniform(0, 6)), m))
    return ops


@pytest.mark.parametrize("n", [1, 2, 3, 5, 7, 10, 12, 13, 14, 15])
@pytest.mark.parametrize("dtype,tol", [("c128", 1e-12), ("c64", 1e-5)])
@pytest.mark.parametrize("fused", [False, True])
def test_small_circuits(n, dtype, tol, fused):
    for count in (2, 47, 130):
        ops = circuit(n, count, 10 * n + count)
        psi0 = W.gaussian_state(n, 60 + n).astype(np.complex128 if dtype == "c128" else np.complex64)
        st = sv.State(n, dtype).load(psi0)
        sv.Circuit(n, ops).apply(st, fuse_diagonal=fused)
        ref = oracle.run_circuit(psi0.astype(np.complex128), ops)
        assert float(np.max(np.abs(st.numpy() - ref))) <= tol


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_moves_are_exact(dtype):
    n = 11
    rng = np.random.default_rng(2)
    ops = []
    for _ in range(60):
        q = [int(x) for x in rng.permutation(n)]
        ops.append(Op("SWAP", (q[2],), (q[0], q[1])) if rng.integers(2) else Op("X", tuple(q[1:1 + int(rng.integers(0, 3))]), (q[0],)))
    psi0 = W.gaussian_state(n, 5).astype(np.complex128 if dtype == "c128" else np.complex64)
    st = sv.State(n, dtype).load(psi0)
    sv.Circuit(n, ops).apply(st)
    assert np.array_equal(st.numpy(), oracle.run_circuit(psi0.copy(), ops))
