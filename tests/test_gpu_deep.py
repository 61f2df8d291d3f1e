"""Launches of more than half a small work item per CU and at most one run with a
ring of four stages (long chains here): every partial block exact (integer-valued inputs) in all
layouts, for full and clipped items, and C with it."""
import numpy as np
import pytest

import paper_2512_22142_amd as cleave
from oracle import gemm as og
from oracle import planner
from workloads.tensors import make_matrix

from gpu_util import GpuGemm, block_of, stored

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("transA,transB", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,steps,S", [
    (1024, 1536, 16, 2),      # 192 full items
    (1000, 2040, 17, 2),      # 256 items, the edges clipped
    (2048, 1304, 19, 1)])     # 176 items, one chunk
def test_deep_ring_exact(M, N, steps, S, transA, transB):
    K = 64 * steps * S
    a = make_matrix(1101, M, K, "bf16", integer_valued=True)
    b = make_matrix(1102, K, N, "bf16", integer_valued=True)
    plan = cleave.plan_uniform(M, N, K, 128, 128, S)
    tasks, _ = planner.plan_uniform(M, N, K, 128, 128, S)
    run = GpuGemm(plan, stored(a, transA), stored(b, transB), transA, transB).run()
    assert "128x128_deep" in plan.last_kernel
    parts, C = run.partials_host(), run.C_host()
    ref = [og.gemm(og.widen(a), og.widen(b), s * K // S, (s + 1) * K // S) for s in range(S)]
    for t in tasks:
        m0, ml, n0, nl = int(t["m0"]), int(t["m_len"]), int(t["n0"]), int(t["n_len"])
        assert np.array_equal(block_of(parts, t), ref[int(t["ksplit_idx"])][m0:m0 + ml, n0:n0 + nl]), int(t["tile_id"])
    assert np.array_equal(C, sum(ref))
