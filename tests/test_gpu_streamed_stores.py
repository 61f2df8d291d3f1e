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
                                           (8192, 8192, torch.float32), (8456, 8192, torch.float32)])
def test_assembled_output_around_the_size_of_the_cache(M, N, out_dtype):
    """256 MiB and a little below or above it, full and clipped sub-tiles; sums below 2^8 in
    magnitude are exact in bf16 too."""
    A, B = ints((M, 64), 1) * (torch.arange(64, device="cuda") < 16), ints((64, N), 2)
    plan = cleave.plan_uniform(M, N, 64, 512, 512, 1)
    C = torch.full((M, N), float("nan"), dtype=out_dtype, device="cuda")
    cleave.execute_assemble(plan, A, B, C)
    assert torch.equal(C.float(), exact(A, B))


@pytest.mark.parametrize("M,N,K,S", [(4096, 5376, 1536, 4), (4096, 4864, 1536, 4), (8192, 6144, 832, 2), (4096, 10752, 3072, 8),
                                     (10240, 10240, 1536, 4)])
def test_partial_blocks_around_the_lines(M, N, K, S):
    """Some, none and all of the chunks streamed; a task issued again writes the same bits."""
    A, B = ints((M, K), 3), ints((K, N), 4)
    plan = cleave.plan_uniform(M, N, K, 512, 512, S)
    parts = torch.full((plan.partial_elems,), float("nan"), dtype=torch.float32, device="cuda")
    cleave.execute(plan, A, B, parts)
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


@pytest.mark.parametrize("N", [10232, 10240])
def test_checked_sum_around_the_line(N):
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
