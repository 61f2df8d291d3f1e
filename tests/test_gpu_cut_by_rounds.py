"""Which launches cut large blocks small: by their rounds of the chip and the length
of their chains, at both sides of every line.  Whichever cut is taken, every block
is where the same tasks issued as a subset, which never cuts so many blocks, put
it, and C equals the fp64 oracle exactly (integer-valued inputs); with real-valued
ones, whose sums depend on their order, the two launches' bits are the same."""
import numpy as np
import pytest
import torch

import paper_2512_22142_amd as cleave
from oracle import gemm as og
from workloads.tensors import make_matrix

from gpu_util import stored

pytestmark = pytest.mark.gpu

LARGE, SMALL = "direct_bf16_256x256", "direct_bf16_128x128"


def check(M, N, K, tile, S, transA, transB, kernel):
    a = make_matrix(M * 3 + K, M, K, "bf16", integer_valued=True)
    b = make_matrix(N * 5 + K, K, N, "bf16", integer_valued=True)
    A, B = stored(a, transA), stored(b, transB)
    plan = cleave.plan_uniform(M, N, K, tile, tile, S)
    parts, again = (torch.full((plan.partial_elems,), float("nan"), device="cuda") for _ in range(2))
    C = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    dA, dB = A.cuda(), B.cuda()
    cleave.execute(plan, dA, dB, parts, transA, transB)
    assert kernel in plan.last_kernel, plan.last_kernel
    cleave.reduce(plan, parts, C)
    cleave.execute(plan, dA, dB, again, transA, transB, task_ids=list(range(plan.num_tasks)))
    assert LARGE in plan.last_kernel, plan.last_kernel
    torch.cuda.synchronize()
    assert torch.equal(parts.view(torch.int32), again.view(torch.int32))
    assert np.array_equal(C.cpu().numpy(), og.gemm(*og.logical_operands(A, transA, B, transB)))


# the lines are drawn for 256 CUs; `rows` blocks of 256 rows times `cols` of 256 columns
@pytest.mark.parametrize("rows,cols,steps,kernel", [
    (16, 12, 4, SMALL), (16, 12, 5, LARGE), (16, 13, 4, LARGE),     # up to three quarters of a round, short chains
    (16, 16, 2, LARGE),                                             # a full round
    (16, 17, 40, SMALL), (16, 18, 20, SMALL),                       # a little over one, any chain
    (16, 19, 16, SMALL), (16, 20, 17, LARGE), (16, 21, 2, LARGE),   # up to a quarter more
    (32, 16, 2, LARGE), (32, 17, 8, SMALL), (32, 17, 9, LARGE),     # a little over two, short chains
    (32, 18, 2, LARGE), (16, 49, 2, LARGE),
])
def test_cut_at_the_lines(rows, cols, steps, kernel):
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the sizes are multiples of 256 CUs")
    check(rows * 256, cols * 256, steps * 64, 256, 1, 0, 0, kernel)


@pytest.mark.parametrize("rows,cols,steps,kernel", [
    (16, 14, 24, SMALL), (16, 14, 25, LARGE), (16, 15, 2, LARGE), (16, 16, 2, LARGE),
    (16, 22, 24, SMALL), (16, 24, 12, SMALL), (16, 24, 13, LARGE), (16, 25, 2, LARGE),
    (16, 36, 24, SMALL), (16, 36, 25, LARGE), (16, 40, 8, SMALL), (16, 40, 9, LARGE), (16, 41, 2, LARGE),
    # less than one small block to eight large ones
    (28, 8, 12, SMALL), (28, 8, 13, LARGE), (24, 8, 24, SMALL), (24, 8, 25, LARGE), (32, 12, 8, SMALL), (32, 12, 9, LARGE),
    (32, 16, 2, LARGE), (32, 17, 16, SMALL), (32, 17, 17, LARGE), (32, 18, 8, SMALL), (32, 18, 9, LARGE),
    (32, 20, 4, SMALL), (32, 20, 5, LARGE), (32, 21, 2, LARGE),
    # more than one to two
    (2, 112, 12, SMALL), (2, 112, 13, LARGE),
])
def test_cut_at_the_lines_with_a_rim_of_small_blocks(rows, cols, steps, kernel):
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the sizes are multiples of 256 CUs")
    check(rows * 256 + 72, cols * 256, steps * 64, 256, 1, 0, 0, kernel)


@pytest.mark.parametrize("transA,transB", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("cols,K,kernel", [(17, 1024, SMALL), (17, 1032, SMALL), (21, 1032, LARGE)])
def test_bits_do_not_depend_on_the_cut(cols, K, kernel, transA, transB):
    M, N = 4096, cols * 256
    a, b = stored(make_matrix(cols, M, K, "bf16"), transA), stored(make_matrix(cols + 1, K, N, "bf16"), transB)
    plan = cleave.plan_uniform(M, N, K, 256, 256, 1)
    parts, again = (torch.full((plan.partial_elems,), float("nan"), device="cuda") for _ in range(2))
    dA, dB = a.cuda(), b.cuda()
    cleave.execute(plan, dA, dB, parts, transA, transB)
    assert kernel in plan.last_kernel, plan.last_kernel
    cleave.execute(plan, dA, dB, again, transA, transB, task_ids=list(range(plan.num_tasks)))
    assert LARGE in plan.last_kernel, plan.last_kernel
    few = torch.full_like(parts, float("nan"))
    cleave.execute(plan, dA, dB, few, transA, transB, task_ids=list(range(100)))     # cut small
    assert SMALL in plan.last_kernel, plan.last_kernel
    torch.cuda.synchronize()
    assert not bool(torch.isnan(parts).any())
    assert torch.equal(parts.view(torch.int32), again.view(torch.int32))
    n = 100 * 256 * 256
    assert torch.equal(parts[:n].view(torch.int32), few[:n].view(torch.int32))


@pytest.mark.parametrize("transA,transB", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_clipped_blocks_members_of_both_classes_and_shorter_last_chunks(transA, transB):
    check(17 * 256 - 104, 16 * 256, 2 * 72, 256, 1, transA, transB, SMALL)
    check(8 * 512 + 8, 8 * 512 + 264, 200, 512, 1, transA, transB, SMALL)    # a rim of small blocks
    if transA and not transB:
        check(8 * 256, 12 * 256, 770, 256, 3, transA, transB, SMALL)         # chunks of 257, 257 and 256


@pytest.mark.parametrize("K,S,every,kernel", [
    (128, 2, 2, SMALL),       # chunks of two steps and of one: no more apart than a shorter last chunk
    (192, 3, 2, LARGE),       # of three steps and of one
    (320, 5, 10, LARGE), (1024, 2, 20, LARGE),
])
def test_only_lists_of_equal_items_are_cut_by_rounds(K, S, every, kernel):
    """A little over a round of large items, some of them shorter: every `every`-th
    tile of the first rows is split in S."""
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the sizes are multiples of 256 CUs")
    ks, items = [], 0
    while len(ks) % 16 or items < 264:       # whole rows of 16 tiles
        ks.append(S if len(ks) % every == 0 and items + S <= 272 else 1)
        items += ks[-1]
    rows = len(ks) // 16
    assert 256 < items <= 288
    M, N = rows * 256, 4096
    plan = cleave.plan_explicit(M, N, K, [256] * rows, [[256] * 16] * rows, ks)
    a = make_matrix(K, M, K, "bf16", integer_valued=True)
    b = make_matrix(K + 1, K, N, "bf16", integer_valued=True)
    parts = torch.full((plan.partial_elems,), float("nan"), device="cuda")
    C = torch.full((M, N), float("nan"), device="cuda")
    cleave.execute(plan, a.cuda(), b.cuda(), parts)
    assert kernel in plan.last_kernel, plan.last_kernel
    cleave.reduce(plan, parts, C)
    torch.cuda.synchronize()
    assert np.array_equal(C.cpu().numpy(), og.gemm(*og.logical_operands(a, 0, b, 0)))


@pytest.mark.parametrize("dtype,K", [("bf16", 512), ("bf16", 1088), ("f32", 512), ("f32", 520)])
def test_cut_small_lists_of_unequal_items(dtype, K):
    """Few large blocks among many small ones whose chunks differ by a factor of
    eight: the all-small list in its balanced order (bf16) and as it was laid out
    (fp32, the general kernel's)."""
    M, N = 4096, 2048
    band_h, col_w = [256] * 16, [[256] + [128] * 14] * 16
    ks = [(1, 2, 4, 8)[(3 * i + j) % 4] for i in range(16) for j in range(15)]
    plan = cleave.plan_explicit(M, N, K, band_h, col_w, ks)
    strided, used = cleave.schedule_loads(plan, 2, 512, False), cleave.schedule_loads(plan, 2, 512, True)
    assert used.max() < strided.max()
    a = make_matrix(K, M, K, dtype, integer_valued=True)
    b = make_matrix(K + 1, K, N, dtype, integer_valued=True)
    dA, dB = a.cuda(), b.cuda()
    parts, again = (torch.full((plan.partial_elems,), float("nan"), device="cuda") for _ in range(2))
    C = torch.full((M, N), float("nan"), device="cuda")
    cleave.execute(plan, dA, dB, parts)
    assert (SMALL if dtype == "bf16" else "execute_f32") in plan.last_kernel, plan.last_kernel
    cleave.reduce(plan, parts, C)
    cleave.execute(plan, dA, dB, again, task_ids=list(range(plan.num_tasks)))
    torch.cuda.synchronize()
    assert torch.equal(parts.view(torch.int32), again.view(torch.int32))
    assert np.array_equal(C.cpu().numpy(), og.gemm(*og.logical_operands(a, 0, b, 0)))
