"""The aggregation's runs of elements: bit for bit the oracle's fp32 left fold
for tiles whose rows are shorter and longer than a run and do not divide it, for
every number of splits with a path of its own and one beyond, through the
vector and the element path, into padded outputs."""
import numpy as np
import pytest
import torch

import paper_2512_22142_amd as cleave
from oracle import gemm as og
from oracle import planner

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S", [1, 2, 3, 4, 5, 8, 9])
@pytest.mark.parametrize("M,N,tm,tn", [
    (97, 1204, 50, 600),        # rows of 600 and 4: runs start anywhere in a row
    (5, 9000, 4, 5000),         # rows longer than any run
    (300, 12, 300, 12),         # many rows per run
    (64, 4096, 64, 1024), (33, 331, 20, 101), (3, 1, 2, 1)])
@pytest.mark.parametrize("pad", [0, 4, 3])
def test_runs_equal_the_left_fold(M, N, tm, tn, S, pad):
    K = 72
    plan = cleave.plan_uniform(M, N, K, tm, tn, S)
    tasks, elems = planner.plan_uniform(M, N, K, tm, tn, S)
    parts = torch.randn(elems, generator=torch.Generator().manual_seed(M + S))
    fold = og.reduce_partials(tasks, parts.numpy(), M, N)
    for dt in (torch.float32, torch.bfloat16):
        wide = torch.full((M, N + pad), float("nan"), dtype=dt, device="cuda")
        cleave.reduce(plan, parts.cuda(), wide[:, :N])
        torch.cuda.synchronize()
        assert torch.equal(wide[:, :N].cpu(), torch.from_numpy(fold).to(dt))
        assert bool(torch.isnan(wide[:, N:].float()).all())


def test_runs_of_a_batched_plan():
    G, M, N, K, S = 6, 40, 84, 64, 4
    plan = cleave.plan_batched(M, N, K, 32, 64, S, G)
    tasks, elems = planner.plan_batched(M, N, K, 32, 64, S, G)
    parts = torch.randn(elems, generator=torch.Generator().manual_seed(5))
    C = torch.empty((G * M, N), device="cuda")
    cleave.reduce_batched(plan, parts.cuda(), C, (3 * M * N, M * N), 3)
    torch.cuda.synchronize()
    for g in range(G):
        mine = tasks[tasks["gemm_id"] == g]
        fold = og.reduce_partials(mine, parts.numpy(), M, N)
        assert np.array_equal(C[g * M:(g + 1) * M].cpu().numpy(), fold)


@pytest.mark.parametrize("M,N,tm,tn,S", [
    (600, 1000, 600, 1000, 4), (301, 1003, 301, 1003, 2), (700, 644, 512, 512, 8),   # records written by the host
    (3001, 3000, 3001, 3000, 4),   # on the device: one tile, 8793 runs, more than a workgroup's threads
    (3100, 3000, 1000, 900, 4),
    (280, 260, 1, 1, 1)])          # 72800 tiles: more than the workgroups
def test_records_of_large_and_of_many_tiles(M, N, tm, tn, S):
    K = 64
    plan = cleave.plan_uniform(M, N, K, tm, tn, S)
    tasks, elems = planner.plan_uniform(M, N, K, tm, tn, S)
    parts = torch.randn(elems, generator=torch.Generator().manual_seed(M + N))
    C = torch.full((M, N), float("nan"), device="cuda")
    cleave.reduce(plan, parts.cuda(), C)
    torch.cuda.synchronize()
    assert np.array_equal(C.cpu().numpy(), og.reduce_partials(tasks, parts.numpy(), M, N))
