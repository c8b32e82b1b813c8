"""Diagonal observables of a few generic terms, on both sides of the rule that picks their kernel.

Against the fp64 oracle, from sizes below a tile to above the rule's largest state, in both dtypes and through the three
entry points; a term list repeated in the allocation-free call gives the same bits.  Bar: the oracle's energy of k
terms of coefficient below 3, each a sum of 2^n products in double, to 1e-12 k (complex64 states are widened exactly).
"""
import numpy as np
import pytest
import torch

import oracle
import workloads as W

pytestmark = pytest.mark.gpu

sv = pytest.importorskip("paper_2508_13615_amd")


def terms(n, m, seed):
    rng = np.random.default_rng(seed)
    t = []
    for _ in range(m):
        w = int(rng.integers(1, min(n, 5) + 1))
        t.append((float(rng.uniform(-3, 3)), "Z" * w, tuple(int(q) for q in rng.permutation(n)[:w])))
    return t


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n", [1, 2, 8, 9, 12, 13, 16, 20, 21])
def test_generic_diagonal_terms(n, dtype):
    psi = W.gaussian_state(n, 90 + n).astype(np.complex128 if dtype == "c128" else np.complex64)
    st = sv.State(n, dtype).load(psi)
    out = torch.zeros(2, dtype=torch.float64, device="cuda")
    for m in (1, 2, 3, 4, 5, 11, 12, 33, 70):
        t = terms(n, m, m)
        ref = oracle.expval_obs(psi.astype(np.complex128), t)
        assert abs(st.expval(t) - ref) <= 1e-12 * m
        st.expval_dev(t, out[:1])
        st.expval_dev_noalloc(t, out[1:])
        torch.cuda.synchronize()
        e = out.cpu().numpy()
        assert abs(e[0] - ref) <= 1e-12 * m and e[0] == e[1]
