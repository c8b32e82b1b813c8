"""Circuit.adjoint_grad with no room for the pass engine's tables.

The call then walks op by op (values as ever) and tries the engine again at the next call: once the memory is free the
circuit runs on the engine, which shows in the gradient partials it keeps.  The engine is made to need much: tiles of
2^6 amplitudes on 27 qubits, so that one pass of 60 parameterised gates has 960 MiB of partials (the runtime may give
back some hundred MiB of its own when memory runs out).
"""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

sv = pytest.importorskip("paper_2508_13615_amd")
Op = W.Op
MiB = 1 << 20


def free_bytes():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def test_a_full_device_is_not_remembered():
    n, k = 27, 60
    ops = [Op(("RX", "RY")[(i // 6) % 2], (), (i % 6,), i) for i in range(k)]
    th = W.uniform_angles(k, 4)
    psi, lam = sv.State(n), sv.State(n)
    circ = sv.Circuit(n, ops, k)
    for m in (2, 20):  # what the first gradient of either form sets up in a process
        sv.Circuit(6, ops[:m], m).adjoint_grad(sv.State(6), sv.State(6), th[:m], W.sum_z(6))
    tuned = sv.tune_engine_get("c128", True)
    sv.tune_engine_set("c128", True, 6, 8)
    filler = []
    try:
        torch.cuda.empty_cache()
        while free_bytes() > 320 * MiB:
            filler.append(torch.empty(min(16384 * MiB, free_bytes() - 256 * MiB), dtype=torch.uint8, device="cuda"))
        left = free_bytes()
        e0, g0 = circ.adjoint_grad(psi, lam, th, W.sum_z(n))
        assert left - free_bytes() < 128 * MiB  # op by op
        filler.clear()
        torch.cuda.empty_cache()
        left = free_bytes()
        e1, g1 = circ.adjoint_grad(psi, lam, th, W.sum_z(n))
        assert left - free_bytes() > 800 * MiB  # the engine's partials
    finally:
        sv.tune_engine_set("c128", True, *tuned)
        filler.clear()
        torch.cuda.empty_cache()
    assert abs(e0 - e1) <= 1e-12 * n
    assert float(np.max(np.abs(g0 - g1))) <= 1e-12 * n
