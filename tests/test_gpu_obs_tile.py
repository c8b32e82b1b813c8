"""Pauli sums evaluated many terms per read of the state (k_obs_tile), against the fp64 oracle.

Sizes around the tile (2^12 amplitudes): states smaller than, equal to and larger than one tile; terms inside the
lowest qubits, across the tile's edge, on the highest qubits, with odd numbers of Y, several on one xmask, xmasks too
wide for a tile (the one-term kernel), and more terms than one pass holds.  Bar: 1e-12 (complex128 and complex64
alike: complex64 amplitudes are widened before any product) per term, the sum over 2^n products of a normalised state.
"""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu

sv = pytest.importorskip("paper_2508_13615_amd")


def chain(n):
    t = []
    for q in range(n - 1):
        t += [(0.5, "XX", (q, q + 1)), (0.4, "YY", (q, q + 1)), (0.75, "ZZ", (q, q + 1))]
    return t + [(0.3, "X", (q,)) for q in range(n)] + [(-0.2, "Y", (q,)) for q in range(n)] + [(0.25, "Z", (0,))]


def scattered(n, count, seed):
    rng = np.random.default_rng(seed)
    t = []
    for _ in range(count):
        k = int(rng.integers(1, min(n, 5) + 1))
        qs = tuple(int(q) for q in rng.permutation(n)[:k])
        t.append((float(rng.normal()), "".join(rng.choice(list("XYZ"), size=k)), qs))
    return t


def wide(n):
    return [(0.7, "X" * n, tuple(range(n))), (0.3, "Y" * n, tuple(range(n))), (1.1, "XZ", (0, n - 1))]


def diagonal(n):
    """70 generic diagonal terms: two passes without off-diagonal terms."""
    rng = np.random.default_rng(n)
    out = []
    for _ in range(70):
        k = int(rng.integers(1, n + 1))
        out.append((float(rng.normal()), "Z" * k, tuple(int(q) for q in rng.permutation(n)[:k])))
    return out


CASES = [(n, f) for n in (1, 2, 3, 4, 9, 10, 11, 12, 13, 15) for f in ("chain", "scattered", "diagonal")]
CASES += [(n, "wide") for n in (12, 13, 14)] + [(14, "many")]


@pytest.mark.parametrize("n,form", CASES)
@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_pauli_sums_around_the_tile(n, form, dtype):
    psi = W.gaussian_state(n, 700 + n).astype(np.complex128 if dtype == "c128" else np.complex64)
    terms = {"chain": chain, "wide": wide, "diagonal": diagonal, "scattered": lambda k: scattered(k, 9, 40 + k),
             "many": lambda k: scattered(k, 150, 9)}[form](n)
    st = sv.State(n, dtype).load(psi)
    ref = oracle.expval_obs(psi.astype(np.complex128), terms)
    got = st.expval(terms)
    assert abs(got - ref) <= 1e-12 * len(terms), (got, ref)
    assert st.expval(terms) == got  # fixed order
