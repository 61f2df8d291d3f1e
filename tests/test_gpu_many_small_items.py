"""Lists of more than 2048 small work items run in patches of 8 x 8 of them: every block is
computed, clipped ones at the edges of the patches too, in full launches and re-issued."""
import numpy as np
import pytest
import torch

import paper_2512_22142_amd as cleave
from oracle import gemm as og
from workloads.tensors import make_matrix

from gpu_util import stored

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,M,N,K,S,transA,transB", [
    ("bf16", 6208, 5960, 72, 1, 0, 0), ("bf16", 6208, 5960, 136, 2, 0, 1), ("bf16", 3080, 6152, 64, 2, 1, 0),
    ("bf16", 6003, 5999, 65, 1, 0, 0), ("f32", 6001, 6100, 33, 1, 0, 1)])
def test_more_than_2048_small_items_exact(dtype, M, N, K, S, transA, transB):
    a = make_matrix(71, M, K, dtype, integer_valued=True)
    b = make_matrix(72, K, N, dtype, integer_valued=True)
    A, B = stored(a, transA), stored(b, transB)
    plan = cleave.plan_uniform(M, N, K, 128, 128, S)
    assert plan.num_tasks > 2048
    dA, dB = A.cuda(), B.cuda()
    parts = torch.full((plan.partial_elems,), float("nan"), dtype=torch.float32, device="cuda")
    again = torch.full_like(parts, float("nan"))
    C = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    cleave.execute(plan, dA, dB, parts, transA, transB)
    cleave.reduce(plan, parts, C)
    cleave.execute(plan, dA, dB, again, transA, transB, task_ids=list(range(plan.num_tasks)))
    torch.cuda.synchronize()
    assert np.array_equal(C.cpu().numpy(), og.gemm(*og.logical_operands(A, transA, B, transB)))
    assert torch.equal(parts.view(torch.int32), again.view(torch.int32))
