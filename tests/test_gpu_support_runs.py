"""The fused engine's zero amplitudes and phase tables, against the fp64 oracle.

A run starts from |0...0>: a pass works on, loads and stores only the amplitudes that earlier gates can have reached,
and the last pass writes the zeros.  Circuits whose gates reach few qubits, all qubits late, or qubits above and below
the tile, in tiles small enough for many passes.  Runs of controlled phases onto one target become tables (bytes of
the tile index, lanes); controls inside the tile, outside it and across a byte of the index, with one and two controls.
Bars: 1e-12 (complex128) and 1e-5 (complex64) per amplitude.  A parameter that is not a number spreads to every
amplitude its gate's dense form would touch, zeros included.
"""
import math

import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu

sv = pytest.importorskip("paper_2508_13615_amd")
Op = W.Op


def few_qubits(n, rng):
    """Support on three qubits only: most of the state stays zero to the end."""
    q = [1, n // 2, n - 1]
    ops = [Op("X", (), (q[2],)), Op("RY", (), (q[0],), -1, 0.7), Op("H", (), (q[1],))]
    return ops + [Op("X", (q[1],), (q[2],)), Op("PHASE", (q[0], q[1]), (q[2],), -1, 0.4), Op("SWAP", (), (q[0], q[2]))]


def ladder(n, rng):
    """GHZ then a second ladder downwards: the support grows pass by pass."""
    ops = [Op("H", (), (0,))] + [Op("X", (q,), (q + 1,)) for q in range(n - 1)]
    ops += [Op("U4", (), (q + 1, q), -1, 0.0, W.haar_unitary(2, rng)) for q in range(n - 2, -1, -1)]
    return ops


def top_first(n, rng):
    ops = [Op("RY", (), (q,), -1, float(rng.uniform(0, 6))) for q in range(n - 1, n // 2, -1)]
    return ops + [Op("RX", (n - 1,), (0,), -1, 1.1), Op("Y", (), (2,)), Op("U2", (0,), (n // 2,), -1, 0.0, W.haar_unitary(1, rng))]


def fourier(n, rng):
    return [Op("RY", (), (q,), -1, float(rng.uniform(0, 6))) for q in range(n)] + W.qft_ops(n)


def two_controls(n, rng):
    """Doubly controlled phases onto two targets: controls in the tile, outside it, and in two bytes of the index."""
    ops = [Op("H", (), (q,)) for q in range(n)]
    for t in (4, n - 1):
        for a in range(n):
            for b in range(a + 1, n, 3):
                if t not in (a, b):
                    ops.append(Op("PHASE", (a, b), (t,), -1, float(rng.uniform(0, 6))))
        ops += [Op("PHASE", (c,), (t,), -1, float(rng.uniform(0, 6))) for c in range(n) if c != t]
        ops += [Op("H", (), (t,)), Op("T", (), (t,)), Op("S", (), (t,))]
    return ops


FORMS = {f.__name__: f for f in (few_qubits, ladder, top_first, fourier, two_controls)}


@pytest.mark.parametrize("form", sorted(FORMS))
@pytest.mark.parametrize("n,tile,apt", [(13, 5, 8), (13, 6, 16), (14, 10, 16), (15, 9, 8), (7, 7, 16), (16, 0, 0)])
@pytest.mark.parametrize("dtype,tol", [("c128", 1e-12), ("c64", 1e-5)])
def test_zero_amplitudes_and_phase_tables(form, n, tile, apt, dtype, tol):
    ops = FORMS[form](n, np.random.default_rng(3))
    ref = oracle.run_circuit(oracle.zero_state(n), ops)
    b = sv.Batch([(n, ops, 0, "sum_z")], dtype=dtype, tile_qubits=tile, amps_per_thread=apt, with_grad=False)
    for _ in range(2):  # a second run starts from the first one's state
        e, _ = b.run([])
        assert float(np.max(np.abs(b.state(0) - ref))) <= tol
    assert abs(e[0] - oracle.expval_obs(ref, W.sum_z(n))) <= tol * n


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_not_a_number_spreads_to_zero_amplitudes(dtype):
    n = 12
    ops = [Op("RY", (), (0,), 0), Op("H", (), (n - 1,))]
    b = sv.Batch([(n, ops, 1, "sum_z")], dtype=dtype, tile_qubits=5, amps_per_thread=8, with_grad=False)
    e, _ = b.run([math.nan])
    assert np.isnan(e[0]) and np.isnan(b.state(0)).all()
    e, _ = b.run([0.3])  # and the next run is whole again
    ref = oracle.run_circuit(oracle.zero_state(n), ops, [0.3])
    assert float(np.max(np.abs(b.state(0) - ref))) <= 1e-6
    assert abs(e[0] - oracle.expval_obs(ref, W.sum_z(n))) <= 1e-5


def second_byte(n, rng, across):
    """One run onto qubit 3 with tiles of qubits 0..4: pairs of controls inside byte 1 of the tile index (qubits 13 and
    up) and inside byte 0, which is a run of tables; with `across`, one pair with a control in each byte, which is not."""
    pairs = [(13, 14), (14, n - 1), (13, n - 1), (5, 9), (6, 12)] + ([(7, 15)] if across else [])
    ops = [Op("RY", (), (q,), -1, float(rng.uniform(0, 6))) for q in range(n)]
    ops += [Op("PHASE", p, (3,), -1, float(rng.uniform(0, 6))) for p in pairs]
    ops += [Op("PHASE", (q,), (3,), -1, float(rng.uniform(0, 6))) for q in range(n) if q != 3]
    return ops + [Op("H", (), (3,))]


@pytest.mark.parametrize("form", ["within", "across", "two_controls", "fourier"])
@pytest.mark.parametrize("n", [16, 17])
@pytest.mark.parametrize("tile,apt", [(5, 8), (6, 16)])
@pytest.mark.parametrize("dtype,tol", [("c128", 1e-12), ("c64", 1e-5)])
def test_tile_indices_of_two_bytes(form, n, tile, apt, dtype, tol):
    rng = np.random.default_rng(4)
    ops = FORMS[form](n, rng) if form in FORMS else second_byte(n, rng, form == "across")
    ref = oracle.run_circuit(oracle.zero_state(n), ops)
    b = sv.Batch([(n, ops, 0, "sum_z")], dtype=dtype, tile_qubits=tile, amps_per_thread=apt, with_grad=False)
    e, _ = b.run([])
    assert float(np.max(np.abs(b.state(0) - ref))) <= tol
    assert abs(e[0] - oracle.expval_obs(ref, W.sum_z(n))) <= tol * n
