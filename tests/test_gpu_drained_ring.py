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

from gpu_util import stored

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
    assert kernel in plan.last_kernel, plan.last_kernel
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
    check(1416, 1536, K, transA, transB, "128x128_deep")
