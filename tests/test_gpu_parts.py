"""Launches of few small work items run as 64 x 64 parts of them, one workgroup
each: every partial block and C exact (integer-valued inputs), for parts that
are full, clipped and empty, chains shorter and longer than the ring of four
stages, all layouts, and for re-issued subsets, whose bits must not change."""
import numpy as np
import pytest
import torch

import paper_2512_22142_amd as cleave
from oracle import gemm as og
from oracle import planner
from workloads.tensors import make_matrix

from gpu_util import GpuGemm, block_of, stored

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("transA,transB", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,tile,steps,S", [
    (64, 64, 64, 1, 1), (8, 8, 8, 2, 1), (128, 128, 128, 3, 2), (328, 200, 128, 4, 2),
    (184, 136, 128, 5, 2), (264, 320, 200, 9, 1), (1024, 1152, 128, 2, 1)])
def test_parts_exact(M, N, tile, steps, S, transA, transB):
    K = 64 * steps * S
    a = make_matrix(1001, M, K, "bf16", integer_valued=True)
    b = make_matrix(1002, K, N, "bf16", integer_valued=True)
    plan = cleave.plan_uniform(M, N, K, tile, tile, S)
    tasks, _ = planner.plan_uniform(M, N, K, tile, tile, S)
    run = GpuGemm(plan, stored(a, transA), stored(b, transB), transA, transB)
    run.partials[:] = float("nan")
    run.run()
    assert "64x64" in plan.last_kernel
    parts, C = run.partials_host(), run.C_host()
    ref = [og.gemm(og.widen(a), og.widen(b), s * K // S, (s + 1) * K // S) for s in range(S)]
    for t in tasks:
        m0, ml, n0, nl = int(t["m0"]), int(t["m_len"]), int(t["n0"]), int(t["n_len"])
        assert np.array_equal(block_of(parts, t), ref[int(t["ksplit_idx"])][m0:m0 + ml, n0:n0 + nl]), int(t["tile_id"])
    assert np.array_equal(C, sum(ref))
    ids = list(range(0, len(tasks), 3))
    run.partials[:] = float("nan")
    run.execute(task_ids=ids)
    again = run.partials_host()
    for i, t in enumerate(tasks):
        same = np.array_equal(block_of(again, t), block_of(parts, t))
        assert same if i in ids else np.isnan(block_of(again, t)).all()


@pytest.mark.parametrize("pad,origin", [(8, 0), (4, 4), (3, 1)])
@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
def test_parts_assembled_exact(dt, pad, origin):
    M, N, K = 392, 328, 320
    a = make_matrix(1011, M, K, "bf16", integer_valued=True)
    b = make_matrix(1012, K, N, "bf16", integer_valued=True)
    plan = cleave.plan_uniform(M, N, K, 128, 128, 1)
    flat = torch.full((M * (N + pad) + origin,), float("nan"), dtype=dt, device="cuda")
    wide = flat[origin:].view(M, N + pad)
    cleave.execute_assemble(plan, a.cuda(), b.cuda(), wide[:, :N])
    assert "64x64" in plan.last_kernel
    torch.cuda.synchronize()
    ref = torch.from_numpy(og.gemm(og.widen(a), og.widen(b))).to(dt)
    assert torch.equal(wide[:, :N].cpu(), ref)
    assert bool(torch.isnan(wide[:, N:].float()).all()) and bool(torch.isnan(flat[:origin].float()).all())


def test_parts_serve_a_batched_plan_exact():
    n_batch, L, d = 3, 192, 64
    x = make_matrix(1021, L, n_batch * d, "bf16", integer_valued=True)
    y = make_matrix(1022, L, n_batch * d, "bf16", integer_valued=True)
    plan = cleave.plan_batched(L, L, d, 128, 128, 1, n_batch)
    C = torch.empty((n_batch * L, L), dtype=torch.float32, device="cuda")
    cleave.execute_assemble(plan, x.cuda(), y.cuda(), C, 0, 1, (0, d), (0, d), (0, L * L), n_batch)
    assert "64x64" in plan.last_kernel
    torch.cuda.synchronize()
    for g in range(n_batch):
        ref = og.gemm(og.widen(x)[:, g * d:(g + 1) * d].copy(), og.widen(y)[:, g * d:(g + 1) * d].T.copy())
        assert np.array_equal(C[g * L:(g + 1) * L].cpu().numpy(), ref)


@pytest.mark.parametrize("M,N,steps", [(1024, 2176, 8), (1280, 2040, 12)])   # 136 and 160 items
def test_more_than_half_an_item_per_cu_is_not_cut_into_parts(M, N, steps):
    K = 64 * steps
    a = make_matrix(1031, M, K, "bf16", integer_valued=True)
    b = make_matrix(1032, K, N, "bf16", integer_valued=True)
    plan = cleave.plan_uniform(M, N, K, 128, 128, 1)
    run = GpuGemm(plan, a, b).run()
    assert plan.last_kernel == "execute_direct_bf16_128x128_deep_nn"
    assert np.array_equal(run.C_host(), og.gemm(og.widen(a), og.widen(b)))
