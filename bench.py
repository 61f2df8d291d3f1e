#!/usr/bin/env python3
"""Benchmark of the sub-GEMM hot path on one MI355X.

A step is one pass of the whole path over one transformer layer's forward and
backward GEMMs: for every GEMM, execute all of its sub-GEMM tasks into the
fp32 partial workspace, then reduce the K-split partials into C.  Inputs,
plans and task tables are resident in HBM before the timed region.

Prints ONE JSON line.  `value` is total GEMM flops of the step divided by the
step's wall time (execute + reduce), `roofline` describes the execute kernel
(bf16 MFMA bound), `reduce_roofline` the aggregation kernel (HBM bound), and
`cpu_baseline` the fp64 oracle timed on the host cores on a bounded sample of
the same tasks.
"""
import argparse
import gc
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_BF16_TFLOPS = 2500.0     # MI355X dense bf16 MFMA
PEAK_F32_TFLOPS = 157.3
PEAK_HBM_GBPS = 8000.0

# HBM-side bytes per launch (average over the 21 launches of a c3 step) from the
# FETCH_SIZE and WRITE_SIZE counter runs summarised under profiles/ (FETCH_SIZE
# scaled by 2.0, WRITE_SIZE by 1.0: what the same counters read for a plain copy
# of known size).  Valid only for the kernel sources they were taken with: the
# digest below (over the files that define the execute and reduce kernels, what they are
# launched with and the work-item order) is checked at run time and the figures are
# dropped on a mismatch.
COUNTER_TRAFFIC = {
    "workload": "c3",
    "sources_sha256": "d19ea50cc69e6403985b8330a80a590db16400bd86602e63d7282ece4232d8b9",
    "execute_bytes_per_launch": (2.0 * 217937 + 388640) * 1024,
    "reduce_bytes_per_launch": (2.0 * 196589 + 97134) * 1024,
}


def kernel_sources_digest():
    import hashlib
    csrc = os.path.join(ROOT, "paper_2512_22142_amd", "csrc")
    h = hashlib.sha256()
    for name in ("api.cpp", "execute.hip", "execute_direct.hip", "kernels.h", "plan.cpp", "plan_internal.h", "reduce.hip", "tile_store.h"):
        with open(os.path.join(csrc, name), "rb") as f:
            h.update(name.encode() + b"\0" + f.read())
    return h.hexdigest()


def measure_layer(cleave, torch, config_name, steps, warmup, group_levels=False):
    """Builds one configuration's resident inputs, plans and workspace, runs
    `warmup` untimed and `steps` timed steps (every GEMM of the layer: execute
    then reduce) and returns the measurements as a dict of local names."""
    from workloads import layer_config, make_gemm_operands
    cfg = layer_config(config_name)
    in_bytes = 2 if cfg.dtype == "bf16" else 4

    # ---- resident inputs, plans, workspace --------------------------------
    cpu, dev = {}, {}
    gemms = []
    for gid, g in enumerate(cfg.gemms):
        A, B = make_gemm_operands(cfg, g, cache=cpu)
        for name, t in ((g.a, A), (g.b, B)):
            if name not in dev:
                dev[name] = t.cuda()
        if config_name == "c4":
            # heterogeneous guillotine tiling with a K-split per tile, drawn per GEMM
            from workloads import draw_explicit_tiling
            from workloads.configs import C4_TILING_SEED
            band_h, col_w, ks = draw_explicit_tiling(g.M, g.N, g.K, C4_TILING_SEED + gid)
            plan = cleave.plan_explicit(g.M, g.N, g.K, band_h, col_w, ks, gemm_id=gid)
        else:
            plan = cleave.plan_uniform(g.M, g.N, g.K, cfg.tile_m, cfg.tile_n, cfg.ksplit, gemm_id=gid)
        plan.upload()
        gemms.append((g, plan, dev[g.a], dev[g.b]))
    # One partial workspace per DAG level (GEMMs of a level are independent and
    # could be in flight together), sized for the largest level and reused.
    level_elems = {}
    for g, plan, _, _ in gemms:
        level_elems[g.level] = level_elems.get(g.level, 0) + plan.partial_elems
    workspace = torch.empty(max(level_elems.values()), dtype=torch.float32, device="cuda")
    outputs = [torch.empty((g.M, g.N), dtype=torch.float32, device="cuda") for g, _, _, _ in gemms]
    slots = []
    used = {}
    for g, plan, _, _ in gemms:
        off = used.get(g.level, 0)
        slots.append(workspace[off:off + plan.partial_elems])
        used[g.level] = off + plan.partial_elems

    stream = torch.cuda.current_stream()

    # Launches of the timed step: one execute and one reduce per GEMM, or, with
    # --group-levels, the GEMMs of a DAG level (independent, dispatched together,
    # Sec. 4.1) that have the same shape and storage form (the Q, K, V
    # projections; gate and up) as one grouped execute and one grouped reduce
    # launch over a shared task list.  Uniform tilings only: c4 draws a
    # different tiling per GEMM.
    grouping = group_levels and config_name != "c4"
    groups, open_group = [], {}
    for i, (g, _, _, _) in enumerate(gemms):
        key = (g.level, g.kind, g.M, g.N, g.K, g.transA, g.transB)
        if grouping and key in open_group and len(open_group[key]) < 8:
            open_group[key].append(i)
        else:
            open_group[key] = [i]
            groups.append(open_group[key])
    launches = []
    level_used = {}
    for members in groups:
        g0 = gemms[members[0]][0]
        if len(members) == 1:
            plan = gemms[members[0]][1]
        else:
            plan = cleave.plan_batched(g0.M, g0.N, g0.K, cfg.tile_m, cfg.tile_n, cfg.ksplit, len(members))
            plan.upload()
        off = level_used.get(g0.level, 0)
        level_used[g0.level] = off + plan.partial_elems
        launches.append({
            "name": "+".join(gemms[i][0].name for i in members), "members": members, "plan": plan,
            "A": [gemms[i][2] for i in members], "B": [gemms[i][3] for i in members],
            "C": [outputs[i] for i in members], "slot": workspace[off:off + plan.partial_elems],
            "transA": g0.transA, "transB": g0.transB,
            "flops": sum(gemms[i][0].flops for i in members),
            "reduce_bytes": sum(gemms[i][1].partial_elems * 4 + gemms[i][0].M * gemms[i][0].N * 4 for i in members),
            "tasks": plan.num_tasks})

    def step(events=None):
        # one event between consecutive launches: the end of one kernel's
        # interval is the start of the next one's
        if events is not None:
            prev = torch.cuda.Event(enable_timing=True)
            prev.record(stream)
        for i, L in enumerate(launches):
            if len(L["members"]) == 1:
                cleave.execute(L["plan"], L["A"][0], L["B"][0], L["slot"], L["transA"], L["transB"])
            else:
                cleave.execute_grouped(L["plan"], L["A"], L["B"], L["slot"], L["transA"], L["transB"])
            if events is not None:
                mid = torch.cuda.Event(enable_timing=True)
                mid.record(stream)
            if len(L["members"]) == 1:
                cleave.reduce(L["plan"], L["slot"], L["C"][0])
            else:
                cleave.reduce_grouped(L["plan"], L["slot"], L["C"])
            if events is not None:
                end = torch.cuda.Event(enable_timing=True)
                end.record(stream)
                events.append((i, prev, mid, end))
                prev = end

    for _ in range(warmup):
        step()
    torch.cuda.synchronize()

    # ---- timed region: exactly K steps -------------------------------------
    events = []
    t_begin = torch.cuda.Event(enable_timing=True)
    t_end = torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    wall0 = time.perf_counter()
    t_begin.record(stream)
    for _ in range(steps):
        step(events)
    t_end.record(stream)
    torch.cuda.synchronize()
    wall = time.perf_counter() - wall0
    gpu_ms = t_begin.elapsed_time(t_end)
    ms_per_step = max(gpu_ms, wall * 1e3) / steps

    exec_ms = [0.0] * len(launches)
    red_ms = [0.0] * len(launches)
    for i, e0, e1, e2 in events:
        exec_ms[i] += e0.elapsed_time(e1)
        red_ms[i] += e1.elapsed_time(e2)
    exec_ms = [x / steps for x in exec_ms]
    red_ms = [x / steps for x in red_ms]
    # each step on its own: first event of the step to its last
    n_g = len(launches)
    step_ms = sorted(events[k * n_g][1].elapsed_time(events[k * n_g + n_g - 1][3]) for k in range(steps))
    step_median = (step_ms[(len(step_ms) - 1) // 2] + step_ms[len(step_ms) // 2]) / 2

    flops = [L["flops"] for L in launches]
    red_bytes = [L["reduce_bytes"] for L in launches]
    total_flops = float(sum(flops))
    exec_total_ms = sum(exec_ms)
    red_total_ms = sum(red_ms)
    exec_tflops = total_flops / (exec_total_ms * 1e-3) / 1e12
    red_gbps = sum(red_bytes) / (red_total_ms * 1e-3) / 1e9
    value = total_flops / (ms_per_step * 1e-3) / 1e12
    peak = PEAK_BF16_TFLOPS if cfg.dtype == "bf16" else PEAK_F32_TFLOPS
    counters_valid = (config_name == COUNTER_TRAFFIC["workload"] and not grouping and
                      kernel_sources_digest() == COUNTER_TRAFFIC["sources_sha256"])
    exec_traffic = round(COUNTER_TRAFFIC["execute_bytes_per_launch"]) if counters_valid else None
    red_traffic = round(COUNTER_TRAFFIC["reduce_bytes_per_launch"]) if counters_valid else None

    return dict(locals())


def device_state_under_load(torch, step, seconds=0.6, period=0.01):
    """Median board power and reported shader clock while `step` runs back to
    back; None where the driver does not expose the file."""
    import glob
    import statistics
    import threading
    import time

    def first(pattern):
        found = sorted(glob.glob(pattern))
        return found[0] if found else None

    power_file = first("/sys/class/drm/card*/device/hwmon/hwmon*/power1_input") or first(
        "/sys/class/drm/card*/device/hwmon/hwmon*/power1_average")
    cap_file = first("/sys/class/drm/card*/device/hwmon/hwmon*/power1_cap")
    sclk_file = first("/sys/class/drm/card*/device/pp_dpm_sclk")
    power, sclk = [], []
    stop = threading.Event()

    def sample():
        while not stop.is_set():
            try:
                if power_file:
                    power.append(int(open(power_file).read()) / 1e6)
                if sclk_file:
                    cur = [l for l in open(sclk_file).read().splitlines() if l.rstrip().endswith("*")]
                    if cur:
                        sclk.append(float(cur[0].split(":")[1].lower().replace("mhz", "").replace("*", "")))
            except (OSError, ValueError, IndexError):
                pass
            time.sleep(period)

    for _ in range(3):                   # the clock governor reacts within tens of milliseconds
        step()
    torch.cuda.synchronize()
    t = threading.Thread(target=sample)
    t0 = time.time()
    t.start()
    while time.time() - t0 < seconds:
        for _ in range(4):
            step()
        torch.cuda.synchronize()
    stop.set()
    t.join()
    # the first samples still see the ramp: keep the later two thirds
    power, sclk = power[len(power) // 3:], sclk[len(sclk) // 3:]
    cap = None
    try:
        cap = int(open(cap_file).read()) / 1e6 if cap_file else None
    except (OSError, ValueError):
        pass
    return {
        "board_power_w_median": round(statistics.median(power), 1) if power else None,
        "board_power_cap_w": cap,
        "reported_sclk_mhz_median": round(statistics.median(sclk), 1) if sclk else None,
        "nominal_sclk_mhz": 2400,
        "samples": len(power),
        "source": "sysfs hwmon power1_input / pp_dpm_sclk, sampled every %d ms while the step repeats" % int(period * 1e3),
        "note": "roofline.peak assumes the nominal clock",
    }


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--config", default="c3", choices=["c1", "c2", "c3", "c4", "c5"])
    ap.add_argument("--group-levels", action="store_true",
                    help="one grouped launch per set of same-shape GEMMs of a DAG level (12 launches "
                         "per c3 step instead of 21); measured: execute +1 %, reduce -3 %, step time equal")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-graph", action="store_true", help="skip the HIP-graph replay of the step")
    ap.add_argument("--no-verify", action="store_true", help="skip the returned-block check leg")
    ap.add_argument("--no-attention", action="store_true", help="skip the batched attention-product leg")
    ap.add_argument("--no-epilogues", action="store_true", help="skip the fused Adam / residual leg")
    ap.add_argument("--no-other-configs", action="store_true",
                    help="skip the short runs of the other benchmark configurations")
    ap.add_argument("--other-steps", type=int, default=5)
    ap.add_argument("--no-device-state", action="store_true",
                    help="skip the sampling of board power and reported clock while the step runs")
    ap.add_argument("--cpu-seconds", type=float, default=15.0)
    ap.add_argument("--copy-calibration", action="store_true",
                    help="run only a plain 1 GiB device-to-device copy, 10 times (reference "
                         "reading for the FETCH_SIZE / WRITE_SIZE counters) and exit")
    args = ap.parse_args()
    if args.gpus != 1:
        sys.exit("bench.py: this path runs on one GPU only (tasks are independent and would "
                 "shard by output tile without any exchange); run with --gpus 1")

    import numpy as np
    import torch

    from paper_2512_22142_amd.build import ensure_built
    ensure_built()                      # uses the built library; builds only if there is none
    import paper_2512_22142_amd as cleave
    if not torch.cuda.is_available():
        sys.exit("bench.py: no GPU visible")
    torch.cuda.set_device(0)
    if args.copy_calibration:
        src = torch.empty(1 << 28, dtype=torch.float32, device="cuda").normal_()
        dst = torch.empty_like(src)
        for _ in range(10):
            dst.copy_(src)
        torch.cuda.synchronize()
        print(json.dumps({"copy_bytes_read": src.numel() * 4, "copy_bytes_written": src.numel() * 4,
                          "launches": 10}))
        return
    m = measure_layer(cleave, torch, args.config, args.steps, args.warmup, args.group_levels)
    (cfg, in_bytes, cpu, gemms, launches, workspace, slots, outputs, stream, step, grouping) = (
        m[k] for k in ("cfg", "in_bytes", "cpu", "gemms", "launches", "workspace", "slots", "outputs",
                       "stream", "step", "grouping"))
    (ms_per_step, step_median, step_ms, exec_ms, red_ms, flops, red_bytes, total_flops, exec_total_ms,
     red_total_ms, exec_tflops, red_gbps, value, peak, exec_traffic, red_traffic) = (
        m[k] for k in ("ms_per_step", "step_median", "step_ms", "exec_ms", "red_ms", "flops", "red_bytes",
                       "total_flops", "exec_total_ms", "red_total_ms", "exec_tflops", "red_gbps", "value",
                       "peak", "exec_traffic", "red_traffic"))

    per_launch = [{"gemms": L["name"], "tasks": L["tasks"], "kernel": L["plan"].last_kernel,
                   "execute_ms": round(exec_ms[i], 4), "execute_tflops": round(flops[i] / exec_ms[i] / 1e9, 1),
                   "reduce_ms": round(red_ms[i], 4), "reduce_gbps": round(red_bytes[i] / red_ms[i] / 1e6, 1)}
                  for i, L in enumerate(launches)]

    result = {
        "metric": "sub-GEMM task TFLOP/s (layer fwd+bwd, execute + reduce)",
        "value": round(value, 2),
        "unit": "TFLOP/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms_per_step, 4),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": cfg.dtype,
        "data": "synthetic",
        "config": {
            "workload": ("%s: layer fwd+bwd, %d GEMMs in %d launches, %d tasks, " % (
                cfg.name, len(gemms), len(launches), sum(p.num_tasks for _, p, _, _ in gemms))) + (
                "heterogeneous tiles (edges 128..1024), K-split 1..8 per tile" if args.config == "c4" else
                "uniform %dx%d tiles, K-split %d" % (cfg.tile_m, cfg.tile_n, cfg.ksplit)),
            "tile": [cfg.tile_m, cfg.tile_n], "ksplit": cfg.ksplit, "seed": cfg.seed,
        },
        "layer_fwd_bwd_ms": round(ms_per_step, 4),
        "layer_fwd_bwd_ms_median": round(step_median, 4),
        "layer_fwd_bwd_ms_min": round(step_ms[0], 4),
        "execute_ms": round(exec_total_ms, 4),
        "reduce_ms": round(red_total_ms, 4),
        "execute_tflops": round(exec_tflops, 2),
        "pct_mfma_peak": round(100.0 * exec_tflops / peak, 2),
        "reduce_gbps": round(red_gbps, 1),
        "pct_hbm_peak": round(100.0 * red_gbps / PEAK_HBM_GBPS, 2),
        "roofline": {
            "kernel": "execute", "bound": "mfma",
            "achieved": round(exec_tflops, 2), "peak": peak, "unit": "TFLOP/s",
            "frac": round(exec_tflops / peak, 4), "traffic": exec_traffic,
            "traffic_unit": "HBM-side bytes per launch (counters)",
            "algorithmic_bytes_per_launch_avg": sum(
                (g.M * g.K + g.K * g.N) * in_bytes + plan.partial_elems * 4
                for g, plan, _, _ in gemms) / len(launches),
            "launches_per_step": len(launches),
            "avg_launch_ms": round(exec_total_ms / len(launches), 4),
            "flops_per_launch_avg": total_flops / len(launches),
        },
        "reduce_roofline": {
            "kernel": "reduce", "bound": "hbm",
            "achieved": round(red_gbps, 1), "peak": PEAK_HBM_GBPS, "unit": "GB/s",
            "frac": round(red_gbps / PEAK_HBM_GBPS, 4), "traffic": red_traffic,
            "avg_launch_ms": round(red_total_ms / len(launches), 4),
            "bytes_per_launch_avg": sum(red_bytes) / len(launches),
        },
        "per_launch": per_launch,
        "paper_context": "paper reports cost-model times only (e.g. LLaMA-13B fwd GEMMs 0.063 s/step "
                         "at A100 peak rate, Table 2); no measured kernel numbers",
    }

    # ---- the same step replayed from a HIP graph (information: launch gaps) ----
    if not args.no_graph:
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            step()
        for _ in range(max(1, args.warmup)):
            graph.replay()
        g0, g1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        g0.record(stream)
        for _ in range(args.steps):
            graph.replay()
        g1.record(stream)
        torch.cuda.synchronize()
        graph_ms = g0.elapsed_time(g1) / args.steps
        result["hip_graph"] = {"ms_per_step": round(graph_ms, 4),
                               "tflops": round(total_flops / (graph_ms * 1e-3) / 1e12, 2),
                               "note": "the %d launches of a step captured once and replayed; `value` is the "
                                       "eager figure" % (2 * len(launches))}
        del graph

    # ---- board power and reported clock while the step runs (information) -----
    # Sampled from the driver's sysfs files in a thread of this process, over
    # untimed repetitions of the step behind the timed region.
    if not args.no_device_state:
        result["device_state"] = device_state_under_load(torch, step)

    # ---- returned-block check (outside the timed step; reported on its own) -
    if not args.no_verify:
        from workloads import make_probe_vectors
        probes, outs = [], []
        for i, (g, plan, _, _) in enumerate(gemms):
            r, s = make_probe_vectors(cfg.seed * 100 + i, g.M, g.N)
            probes.append((r.cuda(), s.cuda()))
            outs.append(torch.empty(plan.num_tasks, dtype=torch.int32, device="cuda"))
        ver_ms = [0.0] * len(gemms)
        fused_ms = [0.0] * len(gemms)
        reps = max(3, args.steps // 4)
        for rep in range(reps + 1):                      # first pass: warm-up (allocates the plan's scratch)
            for i, (g, plan, dA, dB) in enumerate(gemms):
                cleave.execute(plan, dA, dB, slots[i], g.transA, g.transB)
                e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                e0.record(stream)
                cleave.verify(plan, dA, dB, slots[i], probes[i][0], probes[i][1], 1e-6, outs[i],
                              transA=g.transA, transB=g.transB)
                e1.record(stream)
                torch.cuda.synchronize()
                if rep > 0:
                    ver_ms[i] += e0.elapsed_time(e1) / reps
        accepted = sum(int(o.sum().item()) for o in outs)
        # the check and the aggregation in one pass over the partial blocks
        for rep in range(reps + 1):
            for i, (g, plan, dA, dB) in enumerate(gemms):
                cleave.execute(plan, dA, dB, slots[i], g.transA, g.transB)
                e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                e0.record(stream)
                cleave.verify_reduce(plan, dA, dB, slots[i], probes[i][0], probes[i][1], 1e-6, outs[i],
                                     outputs[i], transA=g.transA, transB=g.transB)
                e1.record(stream)
                torch.cuda.synchronize()
                if rep > 0:
                    fused_ms[i] += e0.elapsed_time(e1) / reps
        fused_accepted = sum(int(o.sum().item()) for o in outs)
        ver_bytes = [plan.partial_elems * 4 + (g.M * g.K + g.K * g.N) * in_bytes + (g.M + g.N) * 4
                     for g, plan, _, _ in gemms]
        ver_gbps = sum(ver_bytes) / (sum(ver_ms) * 1e-3) / 1e9
        result["verify_roofline"] = {
            "kernel": "verify (projections + bilinear form + verdict)", "bound": "hbm",
            "achieved": round(ver_gbps, 1), "peak": PEAK_HBM_GBPS, "unit": "GB/s",
            "frac": round(ver_gbps / PEAK_HBM_GBPS, 4), "traffic": None,
            "ms_per_layer": round(sum(ver_ms), 4),
            "bytes_per_call_avg": sum(ver_bytes) / len(gemms),
            "tasks_accepted": accepted, "tasks": sum(p.num_tasks for _, p, _, _ in gemms),
            "note": "blocks written by execute, tol 1e-6; not part of the timed step",
        }
        fused_bytes = [b + g.M * g.N * 4 for b, (g, _, _, _) in zip(ver_bytes, gemms)]
        fused_gbps = sum(fused_bytes) / (sum(fused_ms) * 1e-3) / 1e9
        result["verify_reduce_roofline"] = {
            "kernel": "verify + reduce fused (projections + per-tile bilinear forms and fold + verdict)",
            "bound": "hbm", "achieved": round(fused_gbps, 1), "peak": PEAK_HBM_GBPS, "unit": "GB/s",
            "frac": round(fused_gbps / PEAK_HBM_GBPS, 4), "traffic": None,
            "ms_per_layer": round(sum(fused_ms), 4),
            "separate_calls_ms_per_layer": round(sum(ver_ms) + red_total_ms, 4),
            "bytes_per_call_avg": sum(fused_bytes) / len(gemms),
            "tasks_accepted": fused_accepted,
            "note": "every partial block read once for its check and for the sum; not part of the timed step",
        }

    # ---- attention products of the same layer as one batched task list each --
    # (outside the timed step; reported on its own).  4 sequences x 32 heads of
    # 1024 x 128 x 1024 score GEMMs for c3, then P V; K = 128 cannot be split.
    if not args.no_attention and args.config in ("c3", "c5"):
        T = cfg.gemms[0].M
        hidden = cfg.gemms[0].K
        s_len, d = 1024, 128
        n_seq, H = T // s_len, hidden // d
        G = n_seq * H
        gen = torch.Generator(device="cpu")
        gen.manual_seed(cfg.seed + 17)
        Q, Kt, V = (torch.randn((T, hidden), generator=gen, dtype=torch.float32).to(torch.bfloat16).cuda()
                    for _ in range(3))
        ld = hidden
        tile = cfg.tile_m
        sp = cleave.plan_batched(s_len, s_len, d, tile, tile, 1, G)
        pv = cleave.plan_batched(s_len, d, s_len, tile, d, cfg.ksplit, G)
        sp.upload()
        pv.upload()
        ws = workspace[:max(sp.partial_elems, pv.partial_elems)] if workspace.numel() >= max(
            sp.partial_elems, pv.partial_elems) else torch.empty(max(sp.partial_elems, pv.partial_elems),
                                                                 dtype=torch.float32, device="cuda")
        P = torch.empty((G * s_len, s_len), dtype=torch.bfloat16, device="cuda")
        O = torch.empty((T, hidden), dtype=torch.float32, device="cuda")
        pv1 = cleave.plan_batched(s_len, d, s_len, tile, d, 1, G)
        pv1.upload()
        sc_strides = (H * s_len * s_len, s_len * s_len)
        tok_strides = (s_len * ld, d)
        # the path: both products without K-split, blocks assembled straight into their outputs
        legs = [
            ("scores.assemble", lambda: cleave.execute_assemble(sp, Q, Kt, P, 0, 1, tok_strides, tok_strides, sc_strides, H),
             2.0 * G * s_len * s_len * d, 2 * T * hidden * 2 + G * s_len * s_len * 2),
            ("pv.assemble", lambda: cleave.execute_assemble(pv1, P, V, O, 0, 0, sc_strides, tok_strides, tok_strides, H),
             2.0 * G * s_len * s_len * d, G * s_len * s_len * 2 + T * hidden * 2 + T * hidden * 4),
        ]
        # for comparison: the same products through fp32 partial blocks and the reducer
        two_call = [
            ("scores.execute", lambda: cleave.execute_batched(sp, Q, tok_strides, Kt, tok_strides, H, ws, 0, 1),
             2.0 * G * s_len * s_len * d, 2 * T * hidden * 2 + sp.partial_elems * 4),
            ("scores.reduce", lambda: cleave.reduce_batched(sp, ws, P, sc_strides, H),
             0.0, sp.partial_elems * 4 + G * s_len * s_len * 2),
            ("pv.execute", lambda: cleave.execute_batched(pv, P, sc_strides, V, tok_strides, H, ws, 0, 0),
             2.0 * G * s_len * s_len * d, G * s_len * s_len * 2 + T * hidden * 2 + pv.partial_elems * 4),
            ("pv.reduce", lambda: cleave.reduce_batched(pv, ws, O, tok_strides, H),
             0.0, pv.partial_elems * 4 + T * hidden * 4),
        ]
        reps = max(5, args.steps)
        att = []
        for name, fn, fl, by in legs + two_call:
            for _ in range(3):
                fn()
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record(stream)
            for _ in range(reps):
                fn()
            e1.record(stream)
            torch.cuda.synchronize()
            ms = e0.elapsed_time(e1) / reps
            att.append({"leg": name, "ms": round(ms, 4), "tflops": round(fl / ms / 1e9, 1),
                        "gbps": round(by / ms / 1e6, 1), "algorithmic_bytes": by})
        tot_ms = sum(a["ms"] for a in att[:len(legs)])
        tot_by = sum(a["algorithmic_bytes"] for a in att[:len(legs)])
        result["attention_roofline"] = {
            "workload": "%d score GEMMs %dx%dx%d and %d P.V GEMMs %dx%dx%d as batched task lists without "
                        "K-split, blocks assembled into bf16 scores / fp32 output" % (G, s_len, d, s_len, G, s_len, s_len, d),
            "bound": "hbm", "achieved": round(tot_by / tot_ms / 1e6, 1), "peak": PEAK_HBM_GBPS,
            "unit": "GB/s", "frac": round(tot_by / tot_ms / 1e6 / PEAK_HBM_GBPS, 4), "traffic": None,
            "ms": round(tot_ms, 4), "tflops": round(4.0 * G * s_len * s_len * d / tot_ms / 1e9, 1),
            "legs": att[:len(legs)], "kernels": [sp.last_kernel, pv1.last_kernel],
            "through_partials": {"ms": round(sum(a["ms"] for a in att[len(legs):]), 4), "legs": att[len(legs):],
                                 "note": "same products with fp32 partial blocks + reduce (P.V with S=%d)" % cfg.ksplit},
            "note": "K = 128 cannot be split usefully; without a split the aggregation is pure assembly and is "
                    "done by the executor's stores",
        }

    # ---- PS-side streaming operators fused into the aggregation --------------
    # (outside the timed step).  Adam behind every weight-gradient GEMM of the
    # layer, residual add behind the two projections that feed the residual stream.
    if not args.no_epilogues:
        reps = max(5, args.steps)
        adam_ms, adam_bytes, res_ms, res_bytes = 0.0, 0, 0.0, 0
        for i, (g, plan, dA, dB) in enumerate(gemms):
            is_dw = g.name.endswith(".dw")
            is_res = g.name in ("o.fwd", "down.fwd")
            if not (is_dw or is_res):
                continue
            cleave.execute(plan, dA, dB, slots[i], g.transA, g.transB)
            if is_dw:
                w = torch.zeros((g.M, g.N), dtype=torch.float32, device="cuda").normal_(0, 0.02)
                m = torch.zeros_like(w)
                v = torch.zeros_like(w)
                w16 = torch.empty((g.M, g.N), dtype=torch.bfloat16, device="cuda")
                state = {"t": 0}

                def fn():
                    state["t"] += 1
                    cleave.reduce_adam(plan, slots[i], w, m, v, 1e-4, 0.9, 0.95, 1e-8, 0.1, state["t"], w_bf16=w16)
                nbytes = plan.partial_elems * 4 + g.M * g.N * 26
            else:
                resid = torch.zeros((g.M, g.N), dtype=torch.float32, device="cuda").normal_()
                out = torch.empty_like(resid)

                def fn():
                    cleave.reduce_residual(plan, slots[i], resid, out)
                nbytes = plan.partial_elems * 4 + g.M * g.N * 8
            for _ in range(2):
                fn()
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record(stream)
            for _ in range(reps):
                fn()
            e1.record(stream)
            torch.cuda.synchronize()
            ms = e0.elapsed_time(e1) / reps
            if is_dw:
                adam_ms += ms
                adam_bytes += nbytes
            else:
                res_ms += ms
                res_bytes += nbytes
            del fn
        result["epilogue_roofline"] = {
            "kernel": "reduce with fused Adam (7 weight-gradient GEMMs) / fused residual add (o.fwd, down.fwd)",
            "bound": "hbm", "achieved": round(adam_bytes / adam_ms / 1e6, 1), "peak": PEAK_HBM_GBPS,
            "unit": "GB/s", "frac": round(adam_bytes / adam_ms / 1e6 / PEAK_HBM_GBPS, 4), "traffic": None,
            "adam_ms_per_layer": round(adam_ms, 4), "adam_bytes_per_param": 26 + 4 * cfg.ksplit,
            "residual_ms": round(res_ms, 4), "residual_gbps": round(res_bytes / res_ms / 1e6, 1),
            "note": "bytes = 4*S per element of partials + 26 per parameter (fp32 w, m, v read and written, "
                    "bf16 copy written); the gradient is never stored",
        }

    # ---- the other configurations, a few steps each (reported, not `value`) ---
    if not args.no_other_configs:
        others = {}
        for name in ("c1", "c2", "c4", "c5"):
            if name == args.config:
                continue
            o = measure_layer(cleave, torch, name, args.other_steps, 2)
            o_peak = o["peak"]
            others[name] = {
                "workload": o["cfg"].name, "dtype": o["cfg"].dtype, "steps": args.other_steps,
                "gemms": len(o["gemms"]), "tasks": sum(p.num_tasks for _, p, _, _ in o["gemms"]),
                "ms_per_step": round(o["ms_per_step"], 4), "tflops": round(o["value"], 2),
                "execute_ms": round(o["exec_total_ms"], 4), "execute_tflops": round(o["exec_tflops"], 2),
                "execute_frac_mfma_peak": round(o["exec_tflops"] / o_peak, 4),
                "reduce_ms": round(o["red_total_ms"], 4), "reduce_gbps": round(o["red_gbps"], 1),
                "reduce_frac_hbm_peak": round(o["red_gbps"] / PEAK_HBM_GBPS, 4),
            }
            if name == "c1":
                others[name]["note"] = "3 MiB of partials: cache-resident, not an HBM measurement"
            del o
            gc.collect()
            torch.cuda.empty_cache()
        result["other_configs"] = others

    # ---- CPU baseline: the oracle as it stands, bounded sample -------------
    if not args.no_cpu_baseline:
        from oracle import gemm as og
        rng = np.random.default_rng(cfg.seed)
        done_flops, done_tasks = 0.0, 0
        spent = 0.0
        order = rng.permutation(len(gemms))
        gi = 0
        while spent < args.cpu_seconds:
            g, plan, _, _ = gemms[int(order[gi % len(gemms)])]
            gi += 1
            A, B = cpu[g.a], cpu[g.b]
            opA, opB = og.logical_operands(A, g.transA, B, g.transB)   # layout step, untimed
            tasks = plan.tasks
            for t in tasks[rng.permutation(len(tasks))[:4]]:
                t0 = time.perf_counter()
                og.task_block(opA, opB, t)
                spent += time.perf_counter() - t0
                done_flops += 2.0 * int(t["m_len"]) * int(t["n_len"]) * int(t["k_len"])
                done_tasks += 1
                if spent >= args.cpu_seconds:
                    break
        result["cpu_baseline"] = {
            "value": round(done_flops / spent / 1e12, 5), "unit": "TFLOP/s",
            "cores": og.num_threads(), "kind": "oracle",
            "sample": "%d randomly drawn tasks of this workload (%.1f GFLOP) in %.1f s of fp64 "
                      "naive-loop GEMM" % (done_tasks, done_flops / 1e9, spent),
        }

    print(json.dumps(result))


if __name__ == "__main__":
    main()
