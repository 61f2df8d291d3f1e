"""bf16 outputs of the execute kernels' full sub-tiles and of the aggregation,
bit for bit: integer-valued inputs make every sum exact in fp32, so the output
must be the nearest-even rounding of the oracle's value; infinities and NaN in
the inputs must come out as such."""
import numpy as np
import pytest
import torch

import paper_2512_22142_amd as cleave
from oracle import gemm as og
from workloads.tensors import make_matrix

pytestmark = pytest.mark.gpu


def _rounded(ref):
    return torch.from_numpy(ref).to(torch.bfloat16).view(torch.int16).numpy()


# ld pad / origin in elements: rows on 16 bytes, on 8 bytes only, and an origin on 4; the
# sub-tile leaves in 16-byte pieces at all of them
@pytest.mark.parametrize("pad,origin", [(8, 0), (4, 4), (12, 0), (8, 4), (4, 2)])
@pytest.mark.parametrize("tile,steps", [(256, 1), (256, 2), (512, 3), (128, 1), (128, 2), (128, 5)])
def test_assembled_bf16_rounds_and_stays_inside(tile, steps, pad, origin):
    # several work items per workgroup for the short chains, clipped sub-tiles at the right edge
    M, N, K = (4096, 4232, 64 * steps) if steps < 3 else (1024, 1160, 64 * steps)
    a = make_matrix(901 + steps, M, K, "bf16", integer_valued=True)
    b = make_matrix(902 + steps, K, N, "bf16", integer_valued=True)
    b[:, 0] *= 64                                     # sums with more than eight significant bits
    plan = cleave.plan_uniform(M, N, K, tile, tile, 1)
    ld = N + pad
    flat = torch.full((M * ld + origin,), float("nan"), dtype=torch.bfloat16, device="cuda")
    wide = flat[origin:].view(M, ld)
    C = wide[:, :N]
    cleave.execute_assemble(plan, a.cuda(), b.cuda(), C)
    assert "direct" in plan.last_kernel
    torch.cuda.synchronize()
    ref = og.gemm(og.widen(a), og.widen(b))
    assert np.array_equal(C.contiguous().view(torch.int16).cpu().numpy(), _rounded(ref))
    assert bool(torch.isnan(wide[:, N:].float()).all()) and bool(torch.isnan(flat[:origin].float()).all())


@pytest.mark.parametrize("assembled", [True, False])
def test_non_finite_sums_keep_their_class(assembled):
    M = N = 256
    K = 128
    a = make_matrix(911, M, K, "bf16", integer_valued=True)
    b = make_matrix(912, K, N, "bf16", integer_valued=True)
    a[3, 5], a[70, 9], a[200, 1] = float("inf"), float("-inf"), float("nan")
    big = torch.finfo(torch.bfloat16).max
    a[129, :], b[:, 131] = big, big                   # overflows to infinity in fp32 already
    plan = cleave.plan_uniform(M, N, K, 256, 256, 1)
    C = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
    if assembled:
        cleave.execute_assemble(plan, a.cuda(), b.cuda(), C)
    else:
        parts = torch.empty(plan.partial_elems, dtype=torch.float32, device="cuda")
        cleave.execute(plan, a.cuda(), b.cuda(), parts)
        cleave.reduce(plan, parts, C)
    torch.cuda.synchronize()
    got = C.float().cpu()
    ref = a.double() @ b.double()
    cols = torch.arange(N) != 131                     # there fp32 sums overflow either way before an infinity joins
    assert torch.equal(torch.isnan(got)[[3, 70, 200]][:, cols], torch.isnan(ref)[[3, 70, 200]][:, cols])
    inf = torch.isinf(ref[[3, 70]]) & cols
    assert torch.equal(got[[3, 70]][inf].double(), ref[[3, 70]][inf])
    assert got[129, 131] == float("inf")
    rest = torch.ones(M, dtype=torch.bool)
    rest[[3, 70, 129, 200]] = False
    assert torch.equal(got[rest][:, cols], ref[rest][:, cols].to(torch.bfloat16).float())


def test_rounding_of_all_fp32_values_equals_the_integer_form():
    """All 2^32 bit patterns (subnormals, ties, infinities, NaN payloads) through
    the aggregation of a single split, in 64 slices: nearest even by integer
    arithmetic, NaN stays a quiet NaN with the upper bits of its payload.  Both
    the four-element stores and, into rows of odd length, the single ones."""
    M = N = 8192
    plan = cleave.plan_uniform(M, N, 64, M, N, 1)
    C = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
    wide = torch.empty((M, N + 1), dtype=torch.bfloat16, device="cuda")
    for first in range(0, 1 << 32, M * N):
        u = torch.arange(first, first + M * N, dtype=torch.int64, device="cuda")
        want = torch.where((u & 0x7fffffff) > 0x7f800000, (u >> 16) | 0x40, (u + 0x7fff + ((u >> 16) & 1)) >> 16)
        want = (want & 0xffff).to(torch.int16).view(M, N)
        parts = u.to(torch.int32).view(torch.float32)
        del u
        cleave.reduce(plan, parts, C)
        cleave.reduce(plan, parts, wide[:, :N])
        assert torch.equal(C.view(torch.int16), want), hex(first)
        assert torch.equal(wide[:, :N].view(torch.int16), want), hex(first)
