"""The general execute kernel (fp32, and every bf16 operand or chunk the fast
kernel does not take) at the sizes where its loads can go wrong: tile edges and
K tails one element around 16 bytes, a K step and a workgroup tile; leading
dimensions and bases that are only element-aligned; operands that end where
their allocation ends; rows shorter than 16 bytes; both workgroup tiles.
Integer-valued inputs: partial sums stay far below 2^24, so every block and C
equal the fp64 oracle exactly."""
import numpy as np
import pytest
import torch

import paper_2512_22142_amd as cleave
from oracle import gemm as og
from oracle import planner
from workloads.tensors import make_matrix

from gpu_util import block_of, stored

pytestmark = pytest.mark.gpu

LAYOUTS = [(0, 0), (0, 1), (1, 0), (1, 1)]


def tight(t, pad):
    """Device copy whose rows are `pad` elements apart from each other's ends and
    whose storage ends with the last element of the last row."""
    rows, cols = t.shape
    ld = cols + pad
    flat = torch.full(((rows - 1) * ld + cols,), float("nan"), dtype=t.dtype, device="cuda")
    view = flat.as_strided((rows, cols), (ld, 1))
    view.copy_(t)
    return view


def check(M, N, K, tile, S, transA, transB, dtype, pad=0, kernel=None):
    a = make_matrix(M * 7 + K, M, K, dtype, integer_valued=True)
    b = make_matrix(N * 5 + K, K, N, dtype, integer_valued=True)
    A, B = stored(a, transA), stored(b, transB)
    plan = cleave.plan_uniform(M, N, K, *tile, S)
    tasks, elems = planner.plan_uniform(M, N, K, *tile, S)
    parts = torch.full((elems,), float("nan"), dtype=torch.float32, device="cuda")
    C = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    pads = pad if isinstance(pad, tuple) else (pad, pad)
    dA, dB = tight(A, pads[0]), tight(B, pads[1])
    cleave.execute(plan, dA, dB, parts, transA, transB)
    if kernel:
        assert kernel in plan.last_kernel, plan.last_kernel
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
    # a task issued again alone (another cut, another workgroup tile): same bits
    parts2 = torch.full_like(parts, float("nan"))
    ids = [len(tasks) // 2, len(tasks) - 1] if len(tasks) > 1 else [0]
    cleave.execute(plan, dA, dB, parts2, transA, transB, task_ids=sorted(set(ids)))
    torch.cuda.synchronize()
    again = parts2.cpu().numpy()
    for i in set(ids):
        assert np.array_equal(block_of(again, tasks[i]), block_of(host, tasks[i]))


@pytest.mark.parametrize("transA,transB", LAYOUTS)
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_edges_of_loads_steps_and_tiles_exact(dtype, transA, transB):
    step = 64 if dtype == "bf16" else 32
    for K in (step - 1, step + 1, 2 * step, 2 * step + 7, 5 * step - 9):
        check(65, 63, K, (64, 64), 1, transA, transB, dtype, pad=1, kernel="64x64")
    for M, N in ((9, 129), (127, 8), (129, 191), (200, 257)):
        check(M, N, 3 * step + 5, (128, 256), 2, transA, transB, dtype, pad=3, kernel="64x64")
        check(M, N, 97, (96, 100), 3, transA, transB, dtype, pad=0)


@pytest.mark.parametrize("transA,transB", LAYOUTS)
def test_edges_of_the_fp32_tile_of_64_exact(transA, transB):
    """As above with more items than run in quarters of the tile."""
    name = "f32_64x64_" + "nt"[transA] + "nt"[transB]
    for K in (31, 33, 64, 71, 151):
        check(770, 701, K, (128, 128), 1, transA, transB, "f32", pad=1, kernel=name)
    check(1089, 1025, 101, (128, 256), 2, transA, transB, "f32", pad=3, kernel=name)
    check(513, 575, 97, (96, 100), 3, transA, transB, "f32", pad=0, kernel=name)


@pytest.mark.parametrize("transA,transB", LAYOUTS)
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_wide_tiles_exact(dtype, transA, transB):
    # more 128 x 128 work items than the narrow tile is used for, full and clipped ones
    M, N = (1400, 1303) if dtype == "bf16" else (2049, 2055)
    check(M, N, 4 * 75 + 1, (256, 250), 4, transA, transB, dtype, pad=1, kernel="128x128")


@pytest.mark.parametrize("transA,transB", LAYOUTS)
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_wide_tiles_of_several_rounds_exact(dtype, transA, transB):
    # beyond three (bf16, NT), seven (TN) and four (fp32) rounds of the CUs: the tile in four waves
    M, N, K, S = (1400, 1303, 8 * 70 - 3, 8) if dtype == "bf16" else (2049, 2055, 4 * 65 - 1, 4)
    check(M, N, K, (256, 250), S, transA, transB, dtype, pad=1, kernel="128x128")


def test_four_waves_of_two_operands_across_exact():
    """bf16, TN: 1815 items of 261 elements, full and clipped ones."""
    M, N, K = 1400, 1900, 11 * 261 - 5
    a, b = make_matrix(51, M, K, "bf16", integer_valued=True), make_matrix(52, K, N, "bf16", integer_valued=True)
    plan = cleave.plan_uniform(M, N, K, 128, 128, 11)
    parts = torch.full((plan.partial_elems,), float("nan"), dtype=torch.float32, device="cuda")
    C = torch.empty((M, N), dtype=torch.float32, device="cuda")
    cleave.execute(plan, tight(stored(a, 1), 1), tight(b, 3), parts, 1, 0)
    assert plan.num_tasks == 1815 and plan.last_kernel == "execute_bf16_128x128_tn"
    cleave.reduce(plan, parts, C)
    torch.cuda.synchronize()
    assert torch.equal(C.cpu(), (a.double() @ b.double()).float())


@pytest.mark.parametrize("transA,transB", LAYOUTS)
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_rows_shorter_than_a_load_exact(dtype, transA, transB):
    for M, N, K, S in ((1, 1, 1, 1), (3, 2, 5, 5), (2, 300, 70, 2), (130, 3, 65, 1), (40, 50, 6, 2), (5, 7, 100, 3)):
        check(M, N, K, (64, 64), S, transA, transB, dtype)


@pytest.mark.parametrize("transA,transB", LAYOUTS)
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_one_operand_by_elements_the_other_in_wide_loads_exact(dtype, transA, transB):
    E, step = (8, 64) if dtype == "bf16" else (4, 32)
    for short, other, K, pad in ((1, E, E, 0), (E - 1, 63, step - 1, 1), (2, 65, step + 1, 0), (1, 200, 2 * step + 7, 1),
                                 (E - 1, 129, 3 * step, 0)):
        check(short, other, K, (64, 64), 1, transA, transB, dtype, pad)
        check(other, short, K, (128, 64), 1, transA, transB, dtype, pad)
    # rows 32 MiB and more apart in one operand
    far = (1 << 25) // (16 // E) + 3
    check(9, 70, 9, (64, 64), 1, transA, transB, dtype, pad=(far, 1), kernel="element")
    check(70, 9, 9, (64, 64), 1, transA, transB, dtype, pad=(1, far), kernel="element")


@pytest.mark.parametrize("M,N,tile,K", [
    (4096, 4096, (512, 256), 16 * 64 + 8),      # 256 full 256 x 256 items
    (2120, 2176, (136, 136), 17 * 64 - 8)])     # 256 clipped ones
def test_large_items_of_two_k_contiguous_operands_exact(M, N, tile, K):
    """Aligned, the fast kernel's; with rows that are not, the general kernel's 256 x
    256 tile where they are issued as a subset (a full launch cuts them small)."""
    check(M, N, K, tile, 1, 0, 1, "bf16", kernel="direct_bf16_256x256")
    a = make_matrix(M * 7 + K, M, K, "bf16", integer_valued=True)
    b = make_matrix(N * 5 + K, K, N, "bf16", integer_valued=True)
    plan = cleave.plan_uniform(M, N, K, *tile, 1)
    parts = torch.full((plan.partial_elems,), float("nan"), dtype=torch.float32, device="cuda")
    C = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    cleave.execute(plan, tight(a, 1), tight(stored(b, 1), 3), parts, 0, 1, task_ids=list(range(plan.num_tasks)))
    assert plan.last_kernel == "execute_bf16_256x256_nt"
    cleave.reduce(plan, parts, C)
    torch.cuda.synchronize()
    assert np.array_equal(C.cpu().numpy(), og.gemm(*og.logical_operands(a, 0, stored(b, 1), 1)))


def test_large_items_of_a_subset_with_unaligned_rows():
    M, N, K = 2120, 2176, 17 * 64 - 8
    a = make_matrix(31, M, K, "bf16")
    b = make_matrix(32, K, N, "bf16")
    plan = cleave.plan_uniform(M, N, K, 136, 136, 1)
    dA, dB = tight(a, 1), tight(stored(b, 1), 3)
    parts = [torch.full((plan.partial_elems,), float("nan"), device="cuda") for _ in range(2)]
    cleave.execute(plan, dA, dB, parts[0], 0, 1)
    assert "128x128" in plan.last_kernel
    cleave.execute(plan, dA, dB, parts[1], 0, 1, task_ids=list(range(plan.num_tasks)))
    assert "256x256" in plan.last_kernel
    torch.cuda.synchronize()
    assert torch.equal(parts[0].view(torch.int32), parts[1].view(torch.int32))
    assert not bool(torch.isnan(parts[0]).any())


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_general_and_fast_kernel_agree_bit_for_bit(dtype):
    """Real-valued inputs, one call with aligned operands and one with the same
    values one element further on: the bits do not depend on the kernel."""
    M, N, K = 384, 520, 640
    a, b = make_matrix(11, M, K, dtype), make_matrix(12, K, N, dtype)
    plan = cleave.plan_uniform(M, N, K, 256, 128, 2)
    out = []
    for pad in (0, 1):
        wide_a = torch.zeros(M, K + 8, dtype=a.dtype, device="cuda")[:, pad:pad + K]
        wide_a.copy_(a)
        parts = torch.empty(plan.partial_elems, dtype=torch.float32, device="cuda")
        cleave.execute(plan, wide_a, b.cuda(), parts)
        assert ("direct" in plan.last_kernel) == (dtype == "bf16" and pad == 0)
        out.append(parts)
    torch.cuda.synchronize()
    assert torch.equal(out[0].view(torch.int32), out[1].view(torch.int32))
