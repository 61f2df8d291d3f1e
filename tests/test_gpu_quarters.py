"""Few fp32 work items run as 32 x 32 quarters of the 64 x 64 tile (16 x 16 matrix
blocks): the bits of the same tasks in a launch of many, and the oracle's values at the
edges of the tile, of the K step and of the chip's rounds of workgroups."""
import numpy as np
import pytest
import torch

import paper_2512_22142_amd as cleave
from oracle import gemm as og
from workloads.tensors import make_matrix

from gpu_util import TOL, block_of, stored

pytestmark = pytest.mark.gpu

LAYOUTS = [(0, 0), (0, 1), (1, 0), (1, 1)]


@pytest.mark.parametrize("transA,transB", LAYOUTS)
@pytest.mark.parametrize("K", [8, 31, 32, 33, 96, 301])
def test_a_few_tasks_have_the_bits_of_the_full_launch(K, transA, transB):
    M, N = 1309, 761                                   # 11 x 6 tiles, the last ones clipped
    A = stored(make_matrix(21, M, K, "f32"), transA)
    B = stored(make_matrix(22, K, N, "f32"), transB)
    plan = cleave.plan_uniform(M, N, K, 128, 128, 1)
    dA, dB = A.cuda(), B.cuda()
    full = torch.empty(plan.partial_elems, dtype=torch.float32, device="cuda")
    cleave.execute(plan, dA, dB, full, transA, transB)
    # more than one workgroup per CU: not the form that reads ahead, as the quarters do
    assert plan.num_tasks == 66 and plan.last_kernel == "execute_f32_64x64_" + "nt"[transA] + "nt"[transB]
    ids = [0, 5, 17, 60, 65]
    few = torch.full_like(full, float("nan"))
    cleave.execute(plan, dA, dB, few, transA, transB, task_ids=ids)
    assert "quarters" in plan.last_kernel
    torch.cuda.synchronize()
    full, few = full.cpu().numpy(), few.cpu().numpy()
    opA, opB = og.logical_operands(A, transA, B, transB)
    exact = og.gemm(opA, opB)
    for i, t in enumerate(plan.tasks):
        got = block_of(few, t)
        if i not in ids:
            assert np.isnan(got).all()
            continue
        assert np.array_equal(got, block_of(full, t))
        m0, n0 = int(t["m0"]), int(t["n0"])
        ref = exact[m0:m0 + got.shape[0], n0:n0 + got.shape[1]]
        assert og.rel_frobenius(got, ref) <= TOL["f32"]


@pytest.mark.parametrize("transA,transB", LAYOUTS)
@pytest.mark.parametrize("K", [127, 128, 255, 256])
def test_two_quarters_on_a_cu_only_with_longer_chunks(K, transA, transB):
    """Up to 16 items in quarters at any length; beyond, where their fewer products per load
    do not cost more than the shorter chains give."""
    least = 256 if (transA, transB) == (0, 1) else 128
    for N, quarters in ((512, True), (640, K >= least), (1024, K >= least)):    # 16, 20 and 32 items
        A = stored(make_matrix(25, 512, K, "f32", integer_valued=True), transA)
        B = stored(make_matrix(26, K, N, "f32", integer_valued=True), transB)
        plan = cleave.plan_uniform(512, N, K, 256, 256, 1)
        parts = torch.empty(plan.partial_elems, dtype=torch.float32, device="cuda")
        C = torch.empty((512, N), dtype=torch.float32, device="cuda")
        cleave.execute(plan, A.cuda(), B.cuda(), parts, transA, transB)
        assert ("quarters" in plan.last_kernel) == quarters, (N, plan.last_kernel)
        cleave.reduce(plan, parts, C)
        torch.cuda.synchronize()
        assert np.array_equal(C.cpu().numpy(), og.gemm(*og.logical_operands(A, transA, B, transB)))


@pytest.mark.parametrize("transA,transB", LAYOUTS)
@pytest.mark.parametrize("K", [33, 64, 65, 97, 161, 192, 193, 224, 225, 257, 289, 544])   # 2 to 17 steps of 32
def test_steps_that_check_no_edge_and_the_last_ones(K, transA, transB):
    """From seven steps on the quarters run pairs of steps without edge checks: the bits of the
    64 x 64 tile that reads nothing ahead, and nothing read behind the operands (NaN there)."""
    M, N = 1088, 1024
    def placed(x):
        rows, cols = x.shape
        room = torch.full((rows * cols + 4096,), float("nan"))
        room[:rows * cols] = x.reshape(-1)
        return room.cuda()[:rows * cols].view(rows, cols)
    A, B = placed(stored(make_matrix(31, M, K, "f32"), transA)), placed(stored(make_matrix(32, K, N, "f32"), transB))
    plan = cleave.plan_uniform(M, N, K, 64, 64, 1)     # 272 tiles, more than one per CU
    full = torch.empty(plan.partial_elems, dtype=torch.float32, device="cuda")
    cleave.execute(plan, A, B, full, transA, transB)
    assert plan.last_kernel == "execute_f32_64x64_" + "nt"[transA] + "nt"[transB]
    ids = [0, 7, 141, 271]
    few = torch.full_like(full, float("nan"))
    cleave.execute(plan, A, B, few, transA, transB, task_ids=ids)
    assert "quarters" in plan.last_kernel
    torch.cuda.synchronize()
    full, few = full.cpu().numpy(), few.cpu().numpy()
    for i in ids:
        assert np.array_equal(block_of(few, plan.tasks[i]), block_of(full, plan.tasks[i]))


@pytest.mark.parametrize("transA,transB", LAYOUTS)
@pytest.mark.parametrize("dtype,K", [("f32", 224), ("f32", 225), ("f32", 256), ("f32", 289), ("f32", 352), ("bf16", 448), ("bf16", 449),
                                     ("bf16", 512), ("bf16", 577), ("bf16", 713)])
def test_one_tile_per_cu_has_the_bits_of_the_full_launch(dtype, K, transA, transB):
    """7 to 12 K steps; launches that leave a CU one 64 x 64 workgroup read ahead from 8 on."""
    M, N = 1309, 1299                                  # 11 x 11 tiles, the last ones clipped
    def placed(x):                                     # odd row stride, NaN behind the rows
        x = stored(x, 0)
        room = torch.full((x.shape[0], x.shape[1] + 1 + x.shape[1] % 2 * 2), float("nan"), dtype=x.dtype)
        room[:, :x.shape[1]] = x
        return room.cuda()[:, :x.shape[1]]
    A = placed(stored(make_matrix(33, M, K, dtype), transA))
    B = placed(stored(make_matrix(34, K, N, dtype), transB))
    plan = cleave.plan_uniform(M, N, K, 128, 128, 1)
    full = torch.empty(plan.partial_elems, dtype=torch.float32, device="cuda")
    cleave.execute(plan, A, B, full, transA, transB)
    layout = "%s_64x64%%s_%s%s" % (dtype, "nt"[transA], "nt"[transB])
    assert plan.last_kernel == "execute_" + layout % ""
    ids = list(range(81, 121))
    few = torch.full_like(full, float("nan"))
    cleave.execute(plan, A, B, few, transA, transB, task_ids=ids)
    assert plan.last_kernel == "execute_" + layout % ("_lone" if K > 7 * (32 if dtype == "f32" else 64) else "")
    torch.cuda.synchronize()
    full, few = full.cpu().numpy(), few.cpu().numpy()
    for i in ids:
        assert np.array_equal(block_of(few, plan.tasks[i]), block_of(full, plan.tasks[i]))


@pytest.mark.parametrize("out_dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("M,N", [(1, 7), (15, 17), (16, 16), (31, 33), (32, 32), (65, 63)])
def test_assembled_edges_of_the_quarter(M, N, out_dtype):
    K = 40
    A, B = make_matrix(23, M, K, "f32"), make_matrix(24, K, N, "f32")
    plan = cleave.plan_uniform(M, N, K, 128, 128, 1)
    wide = torch.full((M, N + 3), float("nan"), dtype=out_dtype, device="cuda")
    cleave.execute_assemble(plan, A.cuda(), B.cuda(), wide[:, :N])
    parts = torch.empty(plan.partial_elems, dtype=torch.float32, device="cuda")
    cleave.execute(plan, A.cuda(), B.cuda(), parts)
    C = torch.empty((M, N), dtype=out_dtype, device="cuda")
    cleave.reduce(plan, parts, C)
    torch.cuda.synchronize()
    assert torch.equal(wide[:, :N], C) and bool(torch.isnan(wide[:, N:].float()).all())
    # bf16 output: one rounding of a value within the fp32 bar
    assert og.rel_frobenius(C.float().cpu().numpy(), og.gemm(*og.logical_operands(A, 0, B, 0))) <= (TOL["f32"] if out_dtype == torch.float32 else 2.0 ** -8)


@pytest.mark.parametrize("dtype,M,N,K,S,tile", [("bf16", 1025, 1999, 131, 4, 128), ("bf16", 1151, 2175, 67, 4, 128), ("f32", 2100, 2000, 40, 1, 64),
                                                ("f32", 2177, 1921, 33, 1, 64), ("f32", 3000, 4000, 40, 1, 128), ("f32", 3968, 4096, 65, 1, 128),
                                                ("f32", 1270, 3070, 99, 3, 128)])
def test_between_one_and_two_rounds_of_workgroups(dtype, M, N, K, S, tile):
    """Integer-valued inputs: every block exact, whoever computes it."""
    # workgroups against those that the chip holds: two 128 x 128 ones on a CU, four 64 x 64 ones
    rounds = -(-M // 128) * -(-N // 128) * S / (2 * torch.cuda.get_device_properties(0).multi_processor_count)
    assert 1 < rounds * (1 if tile == 128 else 2) <= 2
    g = torch.Generator().manual_seed(5)
    A = torch.randint(-3, 4, (M, K), generator=g).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    B = torch.randint(-3, 4, (K, N), generator=g).to(A.dtype)
    plan = cleave.plan_uniform(M, N, K, 128, 128, S)
    parts = torch.full((plan.partial_elems,), float("nan"), dtype=torch.float32, device="cuda")
    C = torch.empty((M, N), dtype=torch.float32, device="cuda")
    for _ in range(2):
        cleave.execute(plan, A.cuda(), B.cuda(), parts)
        cleave.reduce(plan, parts, C)
    assert plan.last_kernel == "execute_%s_%dx%d_nn" % (dtype, tile, tile)
    torch.cuda.synchronize()
    assert torch.equal(C.cpu(), (A.double() @ B.double()).float())
