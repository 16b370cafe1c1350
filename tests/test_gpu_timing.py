"""GPU: the per-kernel timing of a step whose matrices take the one-pass decomposition and projection."""
import dataclasses

import pytest

import bench
import workloads as WL
from tests.harness import gpu_state, case_from_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mixed", [False, True])
def test_no_bracket_is_faster_than_its_kernels_bytes(mixed):
    """Every bracket's algorithmic bytes take at least their time at 8 TB/s (gradients of 1 GB, so
    that the caches do not hold them): an empty bracket does not pass for Optimizer_M."""
    import torch
    from paper_2609_15037_amd import moara as M
    base = WL.WORKLOADS["llama_300m"]
    spec = base.matrices[0]
    mats = [dataclasses.replace(spec, rows=16384, cols=4096, module=WL.UP)] * 4
    if mixed:   # a rank outside the one-pass kernel's range
        mats = mats + [dataclasses.replace(spec, rows=2048, cols=2048, module=WL.Q)]
    table = [0] * len(base.rank_table)
    table[WL.UP], table[WL.Q] = 64, 512
    wl = dataclasses.replace(base, matrices=tuple(mats), rank_table=tuple(table), block_size=32, moment_dtype="bf16")
    assert bench.one_pass(wl, "bf16") == [True] * 4 + [False] * mixed
    c = case_from_workload(wl)
    st = gpu_state(c)
    W, G = [], []
    for i, (m, n, _) in enumerate(c.shapes):
        W.append(torch.zeros(m, n, dtype=torch.bfloat16, device="cuda"))
        G.append(torch.randn(m, n, device="cuda"))
        M.moara_set_tensor(st, i, M.MOARA_T_P, torch.eye(n, c.ranks[i]).numpy())
    for steps in (2, 5):   # warm up, then count
        M.moara_set_timing(st, steps == 5)
        for _ in range(steps):
            M.moara_step(st, W, G, lr=1e-3)
    torch.cuda.synchronize()
    cost = bench.algorithmic_cost(wl, "bf16", 2, moment_bytes=2)
    for kid, name in ((M.MOARA_KERN_DECOMPOSE, "decompose"), (M.MOARA_KERN_PROJECT, "project"),
                      (M.MOARA_KERN_BACKPROJ, "backproject")):
        brackets, ms = M.moara_kernel_stats(st, kid)
        assert brackets == 5 * (2 if mixed and name == "decompose" else 1), (name, brackets)
        assert ms / 5e3 >= cost[name][0] / 8e12, f"{name}: {cost[name][0]} bytes in {ms / 5:.4f} ms"
