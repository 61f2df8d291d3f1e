"""The fast kernel multiplies with 16 x 16 x 32 matrix instructions, the general one
with 32 x 32 x 16: an element's bits must not depend on that, whatever the inputs --
exponents over most of bf16's range with subnormals among them (sums of every
order of magnitude, cancellation, underflow), infinities and NaN -- nor on the
shape of the fast kernel, nor on whether the chunk ends within a step (which the
fast kernel fills with zeros to 32 elements, the general one to 16).  The general kernel runs the same values one element
further on in memory, where the fast one does not go."""
import pytest
import torch

import paper_2512_22142_amd as cleave

pytestmark = pytest.mark.gpu


def wide_range(rows, cols, seed, special):
    g = torch.Generator().manual_seed(seed)
    t = torch.randn((rows, cols), generator=g)
    t = torch.ldexp(t, torch.randint(-70, 60, (rows, cols), generator=g).float())
    t[::3] = torch.ldexp(t[::3], torch.tensor(-60.0))          # many of these are subnormal in bf16 or zero
    if special:
        t[1, cols // 2], t[rows // 2, 1], t[rows - 2, cols - 1] = float("inf"), float("-inf"), float("nan")
    return t.to(torch.bfloat16)


def beside(t):
    """The same matrix one element further on: no row starts on 16 bytes."""
    flat = torch.zeros(t.numel() + 8, dtype=t.dtype, device="cuda")
    view = flat[1:1 + t.numel()].view(t.shape)
    view.copy_(t)
    return view


def compare(shape, tile, kernel, transA, transB, special):
    M, N, K = shape
    A = wide_range(*((K, M) if transA else (M, K)), 1, special).cuda()
    B = wide_range(*((N, K) if transB else (K, N)), 2, special).cuda()
    plan = cleave.plan_uniform(M, N, K, tile, tile, 1)
    fast, slow = (torch.empty(plan.partial_elems, device="cuda") for _ in range(2))
    cleave.execute(plan, A, B, fast, transA, transB)
    assert kernel in plan.last_kernel, plan.last_kernel
    cleave.execute(plan, beside(A), beside(B), slow, transA, transB)
    assert "direct" not in plan.last_kernel
    nan = torch.isnan(fast)
    assert torch.equal(nan, torch.isnan(slow)) and bool(nan.any()) == special
    assert torch.equal(fast.view(torch.int32)[~nan], slow.view(torch.int32)[~nan])


@pytest.mark.parametrize("special", [False, True])
@pytest.mark.parametrize("transA,transB", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("shape,tile,kernel", [
    ((8192, 5120, 128), 512, "direct_bf16_256x256"),     # several items per workgroup
    ((4352, 2304, 128), 512, "direct_bf16_128x128"),     # large blocks that are cut small
    ((2560, 2560, 192), 128, "direct_bf16_128x128"),
    ((1536, 1408, 1088), 128, "direct_bf16_128x128_deep"),
    ((264, 136, 448), 128, "direct_bf16_64x64"),         # clipped parts
    # chunks that end within a step: 8, 16, 24, 40 and 56 elements of it
    ((8192, 5120, 72), 512, "direct_bf16_256x256"),
    ((8192, 5120, 80), 512, "direct_bf16_256x256"),
    ((4352, 2304, 104), 512, "direct_bf16_128x128"),
    ((2560, 2560, 216), 128, "direct_bf16_128x128"),
    ((1536, 1408, 1080), 128, "direct_bf16_128x128_deep"),
    ((264, 136, 424), 128, "direct_bf16_64x64"),
])
def test_same_bits_from_both_matrix_instructions(shape, tile, kernel, transA, transB, special):
    compare(shape, tile, kernel, transA, transB, special)


@pytest.mark.parametrize("special", [False, True])
@pytest.mark.parametrize("shape,tile,kernel", [
    ((8192, 5120, 65), 512, "direct_bf16_256x256"),
    ((4352, 2304, 131), 512, "direct_bf16_128x128"),
    ((2560, 2560, 177), 128, "direct_bf16_128x128"),
    ((1536, 1408, 1025), 128, "direct_bf16_128x128_deep"),
    ((264, 136, 415), 128, "direct_bf16_64x64"),
])
def test_same_bits_of_odd_chunks(shape, tile, kernel, special):
    compare(shape, tile, kernel, 1, 0, special)
