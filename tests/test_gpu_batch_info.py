"""A batch's info() is what batch_plan said of it, field by field."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

sv = pytest.importorskip("paper_2508_13615_amd")
Op = W.Op


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("grad", [False, True])
@pytest.mark.parametrize("n,tile,apt", [(2, 0, 0), (9, 5, 8), (14, 12, 16), (14, 0, 0)])
@pytest.mark.parametrize("u4", [False, True])
def test_info_is_the_plan(n, tile, apt, dtype, grad, u4):
    ops = W.hea_ops(n, 2)
    if u4:
        ops = ops + [Op("U4", (), (0, 1), -1, 0.0, W.haar_unitary(2, np.random.default_rng(1)))]
    circuits = [(n, ops, W.hea_n_params(n, 2), "sum_z"), (n + 1, W.qft_ops(n + 1), 0, "sum_zz")]
    kw = dict(dtype=dtype, tile_qubits=tile, amps_per_thread=apt, with_grad=grad)
    assert sv.Batch(circuits, **kw).info() == sv.batch_plan(circuits, **kw)
