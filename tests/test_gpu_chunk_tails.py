"""Chunks that end within a K step of the fast kernel, and the forms that its
alignment rules let in: chunks of any length and start where both operands have
the inner dimension across their rows, any number of rows where A's rows run
along it.  Integer-valued inputs: every block and C equal the fp64 oracle
exactly, in all shapes of the kernel, with several items per workgroup, items of
one step, tails in an item's first steps, and unequal chunks."""
import numpy as np
import pytest
import torch

import paper_2512_22142_amd as cleave
from oracle import gemm as og
from oracle import planner
from workloads.tensors import make_matrix

from gpu_util import block_of, stored

pytestmark = pytest.mark.gpu


def layout(transA, transB):
    return "_" + "nt"[transA] + "nt"[transB]


def check(M, N, K, tile, S, transA, transB, kernel=None):
    a = make_matrix(M * 3 + K, M, K, "bf16", integer_valued=True)
    b = make_matrix(N * 5 + K, K, N, "bf16", integer_valued=True)
    A, B = stored(a, transA), stored(b, transB)
    plan = cleave.plan_uniform(M, N, K, *tile, S)
    tasks, elems = planner.plan_uniform(M, N, K, *tile, S)
    parts = torch.full((elems,), float("nan"), dtype=torch.float32, device="cuda")
    C = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    dA, dB = A.cuda(), B.cuda()
    cleave.execute(plan, dA, dB, parts, transA, transB)
    if kernel is None:
        assert "direct_bf16" in plan.last_kernel, plan.last_kernel
    else:
        assert plan.last_kernel == "execute_" + kernel + layout(transA, transB)
    cleave.reduce(plan, parts, C)
    torch.cuda.synchronize()
    opA, opB = og.logical_operands(A, transA, B, transB)
    host = parts.cpu().numpy()
    for s in range(S):
        mine = tasks[tasks["ksplit_idx"] == s]
        ref = og.gemm(opA, opB, int(mine["k0"][0]), int(mine["k0"][0] + mine["k_len"][0]))
        for t in mine:
            m0, ml, n0, nl = int(t["m0"]), int(t["m_len"]), int(t["n0"]), int(t["n_len"])
            assert np.array_equal(block_of(host, t), ref[m0:m0 + ml, n0:n0 + nl]), (M, N, K, int(t["tile_id"]), s)
    assert np.array_equal(C.cpu().numpy(), og.gemm(opA, opB))
    # tasks issued again alone: same bits
    again = torch.full_like(parts, float("nan"))
    ids = sorted({0, len(tasks) // 2, len(tasks) - 1})
    cleave.execute(plan, dA, dB, again, transA, transB, task_ids=ids)
    torch.cuda.synchronize()
    again = again.cpu().numpy()
    for i in ids:
        assert np.array_equal(block_of(again, tasks[i]), block_of(host, tasks[i]))


@pytest.mark.parametrize("transA,transB", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("K,S", [(8, 1), (72, 1), (136, 1), (208, 2), (1104, 3)])
def test_tails_of_whole_eights_exact(K, S, transA, transB):
    check(264, 136, K, (264, 136), S, transA, transB, "direct_bf16_64x64")
    # 221 blocks, then 323: from more than one item per CU on two stages and several items per workgroup
    check(1544, 2056, K, (128, 128), S, transA, transB, "direct_bf16_128x128_deep" if S == 1 else "direct_bf16_128x128")
    if S == 1:
        check(2312, 2056, K, (128, 128), S, transA, transB, "direct_bf16_128x128")
    if S == 1 and K < 200:
        check(8192 + 264, 4608, K, (512, 512), S, transA, transB, "direct_bf16_256x256")   # several items per workgroup
        check(4096 + 264, 4352, K, (512, 512), S, transA, transB, "direct_bf16_128x128")   # a little over a round: cut small


@pytest.mark.parametrize("rows", [15, 16])
def test_a_round_of_large_items_stays_in_the_fast_kernel_beside_tails(rows):
    """About one round of 16-step items of two K-contiguous operands, whole steps,
    in a plan some of whose other chunks end within a step: every launch of it is
    the fast kernel's, the full one and the subset without those."""
    M, N, K = rows * 256, 16 * 256 + 72, 1024
    band_h, col_w, ks = [256] * rows, [[256] * 16 + [72]] * rows, ([1] * 16 + [26]) * rows     # 26 chunks of 40, the last 24
    plan = cleave.plan_explicit(M, N, K, band_h, col_w, ks)
    a = make_matrix(rows, M, K, "bf16", integer_valued=True)
    b = make_matrix(rows + 1, K, N, "bf16", integer_valued=True)
    dA, dB = a.cuda(), stored(b, 1).cuda()
    parts, again = (torch.full((plan.partial_elems,), float("nan"), device="cuda") for _ in range(2))
    C = torch.full((M, N), float("nan"), device="cuda")
    cleave.execute(plan, dA, dB, parts, 0, 1)
    assert "direct" in plan.last_kernel
    cleave.reduce(plan, parts, C)
    ids = [i for i, t in enumerate(plan.tasks) if t["k_len"] == K]
    cleave.execute(plan, dA, dB, again, 0, 1, task_ids=ids)
    assert plan.last_kernel == "execute_direct_bf16_256x256_nt"
    torch.cuda.synchronize()
    assert np.array_equal(C.cpu().numpy(), og.gemm(*og.logical_operands(a, 0, stored(b, 1), 1)))
    host, again = parts.cpu().numpy(), again.cpu().numpy()
    for i in ids:
        assert np.array_equal(block_of(again, plan.tasks[i]), block_of(host, plan.tasks[i]))


def test_tails_in_the_deep_ring_exact():
    for K in (1032, 1080, 1336):
        for transA, transB in ((0, 0), (1, 0), (0, 1)):
            check(1536, 1536, K, (128, 128), 1, transA, transB, "direct_bf16_128x128_deep")


@pytest.mark.parametrize("transA,transB", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K,tile,S,kernel", [
    (8192 + 264, 4608, 136, 512, 1, "direct_bf16_256x256"),
    (4096, 4352, 1032, 512, 1, "direct_bf16_128x128"),     # large blocks cut small
    (1536, 1536, 1080, 128, 1, "direct_bf16_128x128_deep"),
    (1544, 2056, 1104, 128, 3, "direct_bf16_128x128"),
])
def test_tasks_issued_again_have_the_same_bits(M, N, K, tile, S, kernel, transA, transB):
    """Real-valued inputs, whose sums depend on their order: the parts shape, a subset
    with operands one element further on (the general kernel), and the launch of all."""
    a, b = stored(make_matrix(M + K, M, K, "bf16"), transA), stored(make_matrix(N + K, K, N, "bf16"), transB)
    plan = cleave.plan_uniform(M, N, K, tile, tile, S)
    dA, dB = a.cuda(), b.cuda()
    beside = torch.zeros(dA.numel() + 8, dtype=dA.dtype, device="cuda")[1:1 + dA.numel()].view(dA.shape).copy_(dA)
    parts, again, general = (torch.full((plan.partial_elems,), float("nan"), device="cuda") for _ in range(3))
    cleave.execute(plan, dA, dB, parts, transA, transB)
    assert plan.last_kernel == "execute_" + kernel + layout(transA, transB)
    ids = sorted({0, plan.num_tasks // 3, plan.num_tasks // 2, plan.num_tasks - 1})
    cleave.execute(plan, dA, dB, again, transA, transB, task_ids=ids)
    assert "direct_bf16_64x64" in plan.last_kernel, plan.last_kernel
    cleave.execute(plan, beside, dB, general, transA, transB, task_ids=ids)
    assert "direct" not in plan.last_kernel
    torch.cuda.synchronize()
    host, again, general = (x.cpu().numpy().view(np.int32) for x in (parts, again, general))
    for i in ids:
        block = block_of(host, plan.tasks[i])
        assert np.array_equal(block_of(again, plan.tasks[i]), block)
        assert np.array_equal(block_of(general, plan.tasks[i]), block)


@pytest.mark.parametrize("K,S", [(2, 1), (9, 2), (65, 1), (131, 3), (1025, 4)])
def test_any_chunk_of_operands_with_the_inner_dimension_across_their_rows_exact(K, S):
    check(520, 264, K, (264, 136), S, 1, 0)
    check(4096, 2304, K, (512, 512), S, 1, 0)


@pytest.mark.parametrize("M", [1, 3, 127, 1301])
def test_any_number_of_rows_exact(M):
    check(M, 136, 208, (100, 72), 2, 0, 0)
    check(M, 1096, 264, (301, 512), 1, 0, 1)
