"""Re-issue of task subsets (Sec. 4.2, churn recovery) as stream-ordered work:
no host wait, no allocation after the plan's upload, safe on several streams,
and capturable into a HIP graph.  The expected bits are those of the full
launch (a block depends on its own task record only)."""
import numpy as np
import pytest
import torch

import paper_2512_22142_amd as cleave
from workloads import draw_reissue
from workloads.tensors import make_matrix

from gpu_util import GpuGemm

pytestmark = pytest.mark.gpu


def _poison(partials, tasks, ids):
    for i in ids:
        off = int(tasks[i]["partial_off"])
        partials[off:off + int(tasks[i]["m_len"]) * int(tasks[i]["n_len"])] = float("nan")


def _problem(seed=91, M=1024, N=896, K=512, tm=384, tn=256, S=4):
    a = make_matrix(seed, M, K, "bf16")
    b = make_matrix(seed + 1, K, N, "bf16", std=0.02)
    plan = cleave.plan_uniform(M, N, K, tm, tn, S)      # both sub-tile classes, ragged edges
    run = GpuGemm(plan, a, b).execute()
    torch.cuda.synchronize()
    return plan, plan.tasks, run, run.partials.clone()


def test_subset_launch_replays_bitwise_from_a_hip_graph():
    plan, tasks, run, first = _problem()
    lost = draw_reissue(plan.num_tasks, seed=17, fraction=0.3)
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    _poison(run.partials, tasks, lost)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        cleave.execute(plan, run.A, run.B, run.partials, task_ids=lost)
    # replays separated by eager work and synchronisations; every one is checked
    for rep in range(4):
        _poison(run.partials, tasks, lost)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(run.partials.view(torch.int32), first.view(torch.int32)), rep
        # eager subset launches between replays must not disturb the captured one's work list
        other = draw_reissue(plan.num_tasks, seed=100 + rep, fraction=0.5)
        _poison(run.partials, tasks, other)
        cleave.execute(plan, run.A, run.B, run.partials, task_ids=other)
        torch.cuda.synchronize()
        assert torch.equal(run.partials.view(torch.int32), first.view(torch.int32)), rep


def test_captured_subsets_beyond_the_reserved_memory_are_refused():
    plan, tasks, run, first = _problem(seed=93, M=512, N=512, K=256, tm=256, tn=256, S=2)
    every = list(range(plan.num_tasks))
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    refused = None
    with torch.cuda.graph(graph, stream=side):
        cleave.execute(plan, run.A, run.B, run.partials, task_ids=every)       # fills the reserve
        try:
            cleave.execute(plan, run.A, run.B, run.partials, task_ids=every[:1])
        except cleave.CleaveError as e:
            refused = e.status
    assert refused == cleave.ENOMEM
    run.partials.fill_(float("nan"))
    torch.cuda.synchronize()
    graph.replay()
    torch.cuda.synchronize()
    assert torch.equal(run.partials.view(torch.int32), first.view(torch.int32))


def test_subset_launches_on_two_streams_do_not_disturb_each_other():
    plan, tasks, run, first = _problem(seed=95)
    buf = [first.clone(), first.clone()]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    for it in range(24):
        for k in (0, 1):
            lost = draw_reissue(plan.num_tasks, seed=1000 + 2 * it + k, fraction=0.15 + 0.3 * k)
            with torch.cuda.stream(streams[k]):
                _poison(buf[k], tasks, lost)
                cleave.execute(plan, run.A, run.B, buf[k], task_ids=lost)
    torch.cuda.synchronize()
    for k in (0, 1):
        assert torch.equal(buf[k].view(torch.int32), first.view(torch.int32)), k


def test_many_subset_launches_in_flight_wrap_the_work_list_memory():
    plan, tasks, run, first = _problem(seed=97)
    torch.cuda.synchronize()
    # 40 launches of 70 % of the tasks each: far more than the two task lists' worth
    # of work-list memory, enqueued without any synchronisation in between
    for it in range(40):
        lost = draw_reissue(plan.num_tasks, seed=2000 + it, fraction=0.7)
        _poison(run.partials, tasks, lost)
        cleave.execute(plan, run.A, run.B, run.partials, task_ids=lost)
    torch.cuda.synchronize()
    assert torch.equal(run.partials.view(torch.int32), first.view(torch.int32))


@pytest.mark.parametrize("dtype,ld_pad", [("f32", 0), ("bf16", 1), ("bf16", 0)])
def test_captured_subsets_of_large_blocks_take_one_item_per_sub_tile(dtype, ld_pad):
    """The memory set aside for captured calls holds the all-small cut of the task
    list; a subset large enough for the 256 x 256 sub-tiles takes a quarter of it,
    whatever the element type and alignment."""
    M = N = 13 * 136
    K = 64
    plan = cleave.plan_uniform(M, N, K, 136, 136, 1)     # 169 tasks, one 256 x 256 or four 128 x 128 sub-tiles each
    plan.upload()
    g = torch.Generator().manual_seed(322)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    a = torch.randint(-4, 5, (M, K), generator=g).to(torch.float32)
    b = torch.randint(-4, 5, (K, N), generator=g).to(torch.float32)
    dA, dB = a.to(dt).cuda(), torch.zeros((K, N + ld_pad), dtype=dt, device="cuda")[:, :N]
    dB.copy_(b.to(dt))
    want = torch.empty(plan.partial_elems, dtype=torch.float32, device="cuda")
    cleave.execute(plan, dA, dB, want)
    every = list(range(plan.num_tasks))
    bufs = [torch.empty_like(want) for _ in range(4)]
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    refused = []
    with torch.cuda.graph(graph, stream=side):
        for buf in bufs:
            try:
                cleave.execute(plan, dA, dB, buf, task_ids=every)
            except cleave.CleaveError as e:
                refused.append(e.status)
    assert refused == []
    for rep in range(3):
        for buf in bufs:
            buf.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(buf, want) for buf in bufs), rep
