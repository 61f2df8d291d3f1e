"""Lists of blocks smaller than a work item in the general kernel: launched over the
tiles that the largest block of the list fills.  Integer-valued inputs: every block of a
full launch and of a subset equals the oracle exactly, whatever lies beside it."""
import numpy as np
import pytest
import torch

import paper_2512_22142_amd as cleave
from oracle import gemm as og
from workloads.tensors import make_matrix

from gpu_util import block_of, stored

pytestmark = pytest.mark.gpu

# band heights and column widths: all small, one edge small, one larger block among small ones
TILINGS = {
    "64x64": ([64] * 5 + [3], [64] * 6 + [1]),
    "64xmany": ([64, 33, 64], [128, 300, 65]),
    "manyx32": ([200, 128, 7], [32, 17, 32, 31]),
    "one_larger": ([64, 64, 65], [64, 129, 64, 20]),
    "33x97": ([33] * 4, [97] * 3),
}


@pytest.mark.parametrize("transA,transB", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("tiling", list(TILINGS))
def test_blocks_smaller_than_an_item_exact(tiling, dtype, transA, transB):
    heights, widths = TILINGS[tiling]
    M, N, K = sum(heights), sum(widths), 131               # odd: bf16 runs the general kernel too
    n = len(heights) * len(widths)
    plan = cleave.plan_explicit(M, N, K, heights, [widths] * len(heights), [1 + i % 3 for i in range(n)])
    A = stored(make_matrix(41, M, K, dtype, integer_valued=True), transA)
    B = stored(make_matrix(42, K, N, dtype, integer_valued=True), transB)
    opA, opB = og.logical_operands(A, transA, B, transB)
    dA, dB = A.cuda(), B.cuda()
    for ids in (None, list(range(0, plan.num_tasks, 3)), [plan.num_tasks - 1]):
        parts = torch.full((plan.partial_elems,), float("nan"), dtype=torch.float32, device="cuda")
        cleave.execute(plan, dA, dB, parts, transA, transB, task_ids=ids)
        assert "direct" not in plan.last_kernel
        torch.cuda.synchronize()
        got = parts.cpu().numpy()
        for i, t in enumerate(plan.tasks):
            block = block_of(got, t)
            if ids is not None and i not in ids:
                assert np.isnan(block).all()
                continue
            m0, n0, k0 = int(t["m0"]), int(t["n0"]), int(t["k0"])
            ref = og.gemm(opA[m0:m0 + block.shape[0]], opB[:, n0:n0 + block.shape[1]], k0, k0 + int(t["k_len"]))
            assert np.array_equal(block, ref), (i, ids)


@pytest.mark.parametrize("M,N,tile,S,tile_name", [
    (1024, 1024, (64, 64), 2, "64x64"), (2048, 1920, (64, 64), 1, "64x64"), (2048, 1536, (128, 64), 1, "64x64"),   # 512, 960, 384 items
    (2048, 2048, (64, 64), 1, "64x64"), (4096, 2048, (64, 128), 1, "64x64"), (1024, 1024, (32, 32), 1, "64x64"),   # 1024 and more
    (1920, 4096, (128, 128), 1, "128x128"), (3008, 3776, (128, 128), 1, "128x128"), (3072, 3840, (256, 256), 1, "128x128"), (4096, 4096, (128, 128), 1, "128x128")])
def test_items_at_most_half_full_run_in_small_tiles(M, N, tile, S, tile_name):
    """fp32: what counts is the work of the items, not their number (720 items, nearly full
    ones among them: the large tile)."""
    K = 33 * S
    plan = cleave.plan_uniform(M, N, K, *tile, S)
    A = make_matrix(43, M, K, "f32", integer_valued=True).cuda()
    B = make_matrix(44, K, N, "f32", integer_valued=True).cuda()
    parts = torch.full((plan.partial_elems,), float("nan"), dtype=torch.float32, device="cuda")
    C = torch.empty((M, N), dtype=torch.float32, device="cuda")
    cleave.execute(plan, A, B, parts)
    assert plan.last_kernel == "execute_f32_%s_nn" % tile_name
    cleave.reduce(plan, parts, C)
    torch.cuda.synchronize()
    assert torch.equal(C.cpu(), (A.cpu().double() @ B.cpu().double()).float())
