"""lambda = O psi for many Pauli terms in one pass (k_obs_tile_apply), against the fp64 oracle.

Through the adjoint gradient of complex128 circuits: its energy is <psi|lambda>, and the gradients of single rotations
meet lambda on every qubit they touch.  Sizes around the tile (2^12 amplitudes), terms across its edge, odd numbers of
Y, several terms on one xmask, xmasks too wide for a tile, none or only diagonal terms, and more terms than a pass
holds.  The reference gradient is the parameter shift, exact for these gates; bar 1e-12 per term, the sum over 2^n
products of a normalised state.
"""
import math

import numpy as np
import pytest

import oracle
import workloads as W
from test_gpu_obs_tile import chain, diagonal, scattered, wide

pytestmark = pytest.mark.gpu

sv = pytest.importorskip("paper_2508_13615_amd")

FORMS = {"chain": chain, "diagonal": diagonal, "wide": wide, "scattered": lambda n: scattered(n, 9, 60 + n),
         "many": lambda n: scattered(n, 150, 3), "onlywide": lambda n: wide(n)[:2], "lone": lambda n: [(0.9, "Y", (n - 1,))]}
CASES = [(n, f) for n in (1, 2, 3, 9, 11, 12, 13) for f in ("chain", "diagonal", "scattered", "lone")]
CASES += [(13, "wide"), (14, "wide"), (14, "onlywide"), (13, "many")]


@pytest.mark.parametrize("n,form", CASES)
def test_lambda_of_many_terms(n, form):
    psi0 = W.gaussian_state(n, 900 + n)
    terms = FORMS[form](n)
    ops = [W.Op("RY", (), (0,), 0), W.Op("RX", (), (n // 2,), 1), W.Op("RY", (), (n - 1,), 2)]
    th = W.uniform_angles(3, n)
    e, g = sv.Circuit(n, ops, 3).adjoint_grad(sv.State(n).load(psi0), sv.State(n), th, terms)
    bar = 1e-12 * len(terms)
    assert abs(e - oracle.energy(n, ops, th, terms, init=psi0)) <= bar
    for k in range(3):
        s = []
        for d in (0.5, -0.5):
            x = np.array(th, dtype=float)
            x[k] += d * math.pi
            s.append(oracle.energy(n, ops, x, terms, init=psi0))
        assert abs(g[k] - 0.5 * (s[0] - s[1])) <= bar, (k, g[k])
