"""What sv_batch_plan reports for a run, against counts made here (host only)."""
import pytest

import workloads as W

sv = pytest.importorskip("paper_2508_13615_amd")
Op = W.Op


def plan(n, ops, k=0, dtype="c128", grad=False, **shape):
    return sv.batch_plan([(n, ops, k, "sum_z")], dtype, with_grad=grad, **shape)


@pytest.mark.parametrize("dtype,eb", [("c128", 16), ("c64", 8)])
def test_one_pass(dtype, eb):
    n, ops = 8, W.hea_ops(8, 2)
    k = W.hea_n_params(8, 2)
    p = plan(n, ops, k, dtype)
    assert p["passes"] == 1 and p["pass_bytes"] == eb << n  # |0...0> is not loaded, the observable not read
    p = plan(n, ops, k, dtype, grad=True)
    # store; the observable reads psi and writes lambda; the reverse pass reads and writes both
    assert p["passes"] == 1 and p["pass_bytes"] == (1 + 2 + 4) * (eb << n)


def test_zero_amplitudes_are_not_counted():
    n, eb = 12, 16
    ops = [Op("H", (), (q,)) for q in (3, 4)] + [Op("X", (3,), (5,))] + [Op("X", (4,), (6,))]
    p = plan(n, ops, tile_qubits=5, amps_per_thread=8)
    assert p["passes"] == 2
    # two targets of qubits 0..2 and two more each: pass 0 stores its one tile; pass 1 loads the four amplitudes that
    # can hold weight and, as the last, stores the state
    assert p["pass_bytes"] == eb * (2 ** 5 + 2 ** 2 + 2 ** n)
    p = plan(n, ops, grad=True, tile_qubits=5, amps_per_thread=8)
    assert p["pass_bytes"] == eb * (2 ** 5 + 2 ** 2 + (1 + 2 + 8) * 2 ** n)


@pytest.mark.parametrize("name", ["qft", "hea"])
def test_full_size_runs_move_no_more_than_every_pass_whole(name):
    n = 32
    ops, k = (W.qft_ops(n), 0) if name == "qft" else (W.hea_ops(n, 10), W.hea_n_params(n, 10))
    p = plan(n, ops, k)
    sb = 16 << n
    assert sb * (1 if name == "qft" else p["passes"]) <= p["pass_bytes"] <= sb * (2 * p["passes"] - 1)


def test_states_below_a_register_tile_move_whole():
    n = 2  # below 2^3 amplitudes: the observable is a stage of its own
    assert plan(n, [Op("H", (), (0,))])["pass_bytes"] == 2 * (16 << n)


@pytest.mark.parametrize("dtype,tile,grad,u4,expect", [
    ("c128", 12, False, False, 2 ** 11 * 16),  # complex128 forward passes exchange through half a tile
    ("c128", 12, False, True, 2 ** 12 * 16),   # a 4x4 gate sweeps the tile in LDS
    ("c64", 12, False, False, 2 ** 12 * 8),
    ("c128", 10, True, False, 2 ** 10 * 16 + 8 * 64 * 2),  # reverse: a tile and 64 slots of 2 wavefronts
])
def test_lds_bytes(dtype, tile, grad, u4, expect):
    ops = W.hea_ops(14, 1)
    if u4:
        ops = ops + [Op("U4", (), (0, 1), -1, 0.0, [[float(i == j) for j in range(4)] for i in range(4)])]
    p = plan(14, ops, W.hea_n_params(14, 1), dtype, grad=grad, tile_qubits=tile, amps_per_thread=16)
    assert p["lds_bytes"] == expect
