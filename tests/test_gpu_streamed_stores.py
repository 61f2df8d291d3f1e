"""Outputs that the caches cannot hold leave through non-temporal stores: the same bits
in the same places as the plain ones, at sizes on both sides of the rule's lines."""
import pytest
import torch

import paper_2512_22142_amd as cleave

pytestmark = pytest.mark.gpu


def ints(shape, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randint(-3, 4, shape, generator=g, device="cuda").to(torch.bfloat16)


def exact(A, B):
    return (A.double() @ B.double()).float()


@pytest.mark.parametrize("M,N,out_dtype", [(16384, 8192, torch.bfloat16), (16384, 8184, torch.bfloat16),
                                           (8192, 8192, torch.float32), (8456, 8192, torch.float32), (9216, 8192, torch.float32),
                                           (9208, 8192, torch.float32), (18504, 8192, torch.bfloat16)])
def test_assembled_output_around_the_size_of_the_cache(M, N, out_dtype):
    """256 and 288 MiB and a little below or above, full and clipped sub-tiles; sums below 2^8 in
    magnitude are exact in bf16 too."""
    A, B = ints((M, 64), 1) * (torch.arange(64, device="cuda") < 16), ints((64, N), 2)
    plan = cleave.plan_uniform(M, N, 64, 512, 512, 1)
    C = torch.full((M, N), float("nan"), dtype=out_dtype, device="cuda")
    cleave.execute_assemble(plan, A, B, C)
    assert plan.last_kernel == "execute_direct_bf16_256x256_nn"
    assert torch.equal(C.float(), exact(A, B))


@pytest.mark.parametrize("shift,gap,out_dtype", [(0, 8, torch.bfloat16), (1, 1, torch.bfloat16), (3, 5, torch.float32), (0, 0, torch.float32)])
def test_assembled_members_with_gaps_at_any_alignment(shift, gap, out_dtype):
    """257 MiB and more: members `gap` elements further apart than they are long, in rows `gap`
    elements longer than N, from `shift` elements behind an allocation's start."""
    members, inner, L, d = 132, 4, 1024 if out_dtype == torch.bfloat16 else 720, 64
    ld = L + gap
    member = L * ld + gap
    A = ints((members * L, d), 9) * (torch.arange(d, device="cuda") < 16)
    B = ints((members * L, d), 10)
    plan = cleave.plan_batched(L, L, d, 512, 512, 1, members)
    flat = torch.full((shift + members * member + ld,), float("nan"), dtype=out_dtype, device="cuda")
    C = flat[shift:].as_strided((L, L), (ld, 1))
    cleave.execute_assemble(plan, A, B, C, 0, 1, (inner * L * d, L * d), (inner * L * d, L * d), (inner * member, member), inner)
    assert plan.last_kernel == "execute_direct_bf16_256x256_nt"
    assert members * L * L * flat.element_size() >= 256 << 20
    for g in range(members):
        rows = flat[shift + g * member:shift + (g + 1) * member]
        got = rows[:L * ld].view(L, ld)
        a, b = A[g * L:(g + 1) * L], B[g * L:(g + 1) * L]
        assert torch.equal(got[:, :L].float(), exact(a, b.t())), g
        assert bool(torch.isnan(got[:, L:].float()).all()) and bool(torch.isnan(rows[L * ld:].float()).all())
    assert bool(torch.isnan(flat[:shift].float()).all()) and bool(torch.isnan(flat[shift + members * member:].float()).all())


@pytest.mark.parametrize("M,N,K,S", [(4096, 5376, 1536, 4), (4096, 4864, 1536, 4), (8192, 6144, 832, 2), (4096, 10752, 3072, 8),
                                     (10240, 10240, 1536, 4)])
def test_partial_blocks_around_the_lines(M, N, K, S):
    """Some, none and all of the chunks streamed; a task issued again writes the same bits."""
    A, B = ints((M, K), 3), ints((K, N), 4)
    plan = cleave.plan_uniform(M, N, K, 512, 512, S)
    parts = torch.full((plan.partial_elems,), float("nan"), dtype=torch.float32, device="cuda")
    cleave.execute(plan, A, B, parts)
    assert plan.last_kernel == "execute_direct_bf16_256x256_nn"
    C = torch.empty((M, N), dtype=torch.float32, device="cuda")
    cleave.reduce(plan, parts, C)
    assert torch.equal(C, exact(A, B))
    ids = [0, S - 1, plan.num_tasks // 2, plan.num_tasks - 1]
    again = torch.full_like(parts, float("nan"))
    cleave.execute(plan, A, B, again, task_ids=ids)
    for i in ids:
        t = plan.tasks[i]
        a, n = int(t["partial_off"]), int(t["m_len"]) * int(t["n_len"])
        assert torch.equal(again[a:a + n], parts[a:a + n])


@pytest.mark.parametrize("N", [10232, 10240, 11256, 11264, 18424, 18432])
def test_checked_sum_around_the_lines(N):
    M, K = 4096, 128
    A, B = ints((M, K), 5), ints((K, N), 6)
    plan = cleave.plan_uniform(M, N, K, 512, 512, 2)
    parts = torch.empty(plan.partial_elems, dtype=torch.float32, device="cuda")
    cleave.execute(plan, A, B, parts)
    r, s = ints((M,), 7).float(), ints((N,), 8).float()
    accept = torch.empty(plan.num_tasks, dtype=torch.int32, device="cuda")
    forms = [torch.empty(plan.num_tasks, dtype=torch.float64, device="cuda") for _ in range(3)]
    C = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    cleave.verify_reduce(plan, A, B, parts, r, s, 1e-6, accept, C, *forms)
    assert bool(accept.all()) and torch.equal(forms[0], forms[1])
    assert torch.equal(C, exact(A, B))
