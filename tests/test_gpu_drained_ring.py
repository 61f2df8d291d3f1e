"""Launches with one work item (or part of one) per workgroup: the last steps of a chunk
drain the ring of stages, one copy of the step for each number of steps left.  Chunks of
one to ten steps, whole and ending within a step, with integer-valued inputs: every
element of every block equals the fp64 product."""
import numpy as np
import pytest
import torch

import paper_2512_22142_amd as cleave
from oracle import gemm as og
from workloads.tensors import make_matrix

from gpu_util import block_of, stored

pytestmark = pytest.mark.gpu

LAYOUTS = [(0, 0), (0, 1), (1, 0), (1, 1)]


def check(M, N, K, transA, transB, kernel):
    a = make_matrix(61, M, K, "bf16", integer_valued=True)
    b = make_matrix(62, K, N, "bf16", integer_valued=True)
    plan = cleave.plan_uniform(M, N, K, 128, 128, 1)
    parts = torch.full((plan.partial_elems,), float("nan"), dtype=torch.float32, device="cuda")
    C = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    A, B = stored(a, transA), stored(b, transB)
    cleave.execute(plan, A.cuda(), B.cuda(), parts, transA, transB)
    assert plan.last_kernel == "execute_" + kernel + "_" + "nt"[transA] + "nt"[transB]
    cleave.reduce(plan, parts, C)
    torch.cuda.synchronize()
    assert np.array_equal(C.cpu().numpy(), og.gemm(*og.logical_operands(A, transA, B, transB))), (K, transA, transB)


@pytest.mark.parametrize("transA,transB", LAYOUTS)
@pytest.mark.parametrize("steps", range(1, 11))
def test_parts_of_every_number_of_steps_exact(steps, transA, transB):
    for K in (64 * steps, 64 * steps - 8, 64 * steps - 56):
        check(264, 200, K, transA, transB, "direct_bf16_64x64")


@pytest.mark.parametrize("transA,transB", LAYOUTS)
@pytest.mark.parametrize("K", [8, 64, 72, 3 * 64, 4 * 64, 4 * 64 + 8, 5 * 64, 5 * 64 + 24, 9 * 64 - 8, 17 * 64])
def test_deep_ring_exact(K, transA, transB):
    check(1416, 1536, K, transA, transB, "direct_bf16_128x128_deep")


@pytest.mark.parametrize("transA,transB", LAYOUTS)
@pytest.mark.parametrize("bands,kernel", [(2, "direct_bf16_64x64"), (6, "direct_bf16_128x128_deep")])   # 64 and 192 items
def test_whole_chunks_beside_ones_that_end_within_a_step_exact(bands, kernel, transA, transB):
    """17 whole steps, 8.5, 4.25, 2.125 and one in one launch: every block."""
    heights, widths, splits = [128, 104] * (bands // 2), [128, 128, 72, 64, 128], [1, 2, 4, 8, 17]
    M, N, K = sum(heights), sum(widths), 17 * 64
    a = make_matrix(63, M, K, "bf16", integer_valued=True)
    b = make_matrix(64, K, N, "bf16", integer_valued=True)
    plan = cleave.plan_explicit(M, N, K, heights, [widths] * bands, splits * bands)
    assert plan.num_tasks == 32 * bands and {int(t["k_len"]) for t in plan.tasks} == {1088, 544, 272, 136, 64}
    parts = torch.full((plan.partial_elems,), float("nan"), dtype=torch.float32, device="cuda")
    A, B = stored(a, transA), stored(b, transB)
    cleave.execute(plan, A.cuda(), B.cuda(), parts, transA, transB)
    assert plan.last_kernel == "execute_" + kernel + "_" + "nt"[transA] + "nt"[transB]
    torch.cuda.synchronize()
    host = parts.cpu().numpy()
    opA, opB = og.logical_operands(A, transA, B, transB)
    for t in plan.tasks:
        m0, n0, k0 = int(t["m0"]), int(t["n0"]), int(t["k0"])
        block = block_of(host, t)
        ref = og.gemm(opA[m0:m0 + block.shape[0]], opB[:, n0:n0 + block.shape[1]], k0, k0 + int(t["k_len"]))
        assert np.array_equal(block, ref), (int(t["tile_id"]), int(t["ksplit_idx"]))
