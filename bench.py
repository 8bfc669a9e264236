"""Benchmark of the Sketched-SGD hot path on one MI355X.

A step is one pass of the whole path over one batch of W synthetic worker gradients that are
already resident in HBM: W Count-Sketch updates, merge, sketch-space momentum / error
accumulation, estimate of every coordinate, top-k, exact second-round gather, sketch-space
feedback.  Prints ONE JSON line (see the keys below).  Before the inputs are allocated, the
placement step (input_arenas_in_fast_memory) looks for the device memory in which the update runs
fastest against the step's own tables; the same steps are also timed on inputs allocated in
the plain order of a fresh process (`placement.plain_ms_per_step` in the JSON line), and
--plain-placement makes that the only measurement.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--config 4] [--no-cpu-baseline]
                    [--variant V] [--graph] [--plain-placement]
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0          # MI355X published HBM3E peak
METRIC = "sketch+estimate+top-k throughput, Gcoords/s and % HBM peak at d=100M, r=5"
# HBM bytes per launch of the dominant kernel at config 4 (4 launches per step, one per group
# of 8 workers), measured with rocprofv3 --pmc: FETCH_SIZE x 2.000 + WRITE_SIZE x 1.000, the
# factors being what the same counters read for kernels of known traffic in the same run (the
# plain read of one input set, 12.8 GB, and the clearing of the worker tables, 671 MB).
# Source: profiles/accumulate_visits_cfg4_pmc.md.  None for other configs.
MEASURED_TRAFFIC_BYTES = {4: 1.688e10}


def host_cpu():
    """(model name, logical CPUs the process may use, logical CPUs of the machine)"""
    model = "unknown"
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.lower().startswith("model name"):
                    model = line.split(":", 1)[1].strip()
                    break
    except OSError:
        pass
    try:
        usable = len(os.sched_getaffinity(0))
    except AttributeError:
        usable = os.cpu_count() or 1
    return model, usable, os.cpu_count() or usable


def cpu_baseline(cfg, work, sample_acc=64_000_000, sample_est=32_000_000):
    """The CPU reference as it stands, on a bounded sample of the same workload (sized for
    10-30 s of CPU work at config 4), scaled to the cost of one full step.  `value` is one
    thread, which is how the reference is written.  `all_cores` is the same code called from
    several threads at once, one simulated worker's vector (or one slice of the coordinates to
    query) per thread, as independent reference processes would run; the thread count is capped
    at 16, the CPU share of a one-GPU machine, and at the number of workers."""
    import numpy as np
    from concurrent.futures import ThreadPoolExecutor
    from oracle import cs_oracle as orc

    sk = orc.SketchOracle(cfg.r, cfg.c, cfg.hash_seed)
    n_acc = min(sample_acc, cfg.d)
    n_est = min(sample_est, cfg.d)
    g = work.gradient(0, 0)[:n_acc].cpu().numpy()
    t0 = time.perf_counter()
    T = sk.sketch(g)
    t_acc = (time.perf_counter() - t0) / n_acc            # per coordinate of one worker
    t0 = time.perf_counter()
    est = sk.estimate(T, n_est)
    t_est = (time.perf_counter() - t0) / n_est
    k_s = max(1, int(cfg.k * n_est / cfg.d))
    t0 = time.perf_counter()
    orc.topk_threshold(est, k_s)
    t_top = (time.perf_counter() - t0) / n_est
    tabs = [T, T]
    t0 = time.perf_counter()
    orc.merge(tabs)
    t_merge = (time.perf_counter() - t0) / 2 * (cfg.W + (5 if cfg.stateful else 0))
    step_s = cfg.W * cfg.d * t_acc + cfg.d * (t_est + t_top) + t_merge

    model, usable, logical = host_cpu()
    threads = max(1, min(16, usable, cfg.W))
    n_mt = min(n_acc, 16_000_000)
    with ThreadPoolExecutor(max_workers=threads) as pool:
        t0 = time.perf_counter()
        list(pool.map(lambda q: sk.sketch(g[:n_mt]), range(threads)))
        t_acc_mt = (time.perf_counter() - t0) / (threads * n_mt)
        n_est_mt = min(n_est, 8_000_000)
        t0 = time.perf_counter()
        list(pool.map(lambda q: sk.estimate(T, n_est_mt, i0=q * n_est_mt % max(1, cfg.d - n_est_mt)),
                      range(threads)))
        t_est_mt = (time.perf_counter() - t0) / (threads * n_est_mt)
    step_s_mt = cfg.W * cfg.d * t_acc_mt + cfg.d * (t_est_mt + t_top) + t_merge
    return {
        "value": cfg.W * cfg.d / step_s / 1e9,
        "unit": "Gcoords/s",
        "cores": 1,
        "kind": "oracle",
        "sample": (f"update of {n_acc} coords of one worker, estimate+top-k of {n_est} coords, "
                   f"one table merge; scaled to W={cfg.W}, d={cfg.d} (est. {step_s:.1f} s/step)"),
        "all_cores": {"value": cfg.W * cfg.d / step_s_mt / 1e9, "unit": "Gcoords/s", "cores": threads,
                      "sample": (f"{threads} threads at once, each the update of {n_mt} coords of a worker, "
                                 f"then each the estimate of {n_est_mt} coords; selection and merge "
                                 f"single-threaded (est. {step_s_mt:.1f} s/step)")},
        "cpu_model": model,
        "cpus_usable": usable,
        "cpus_logical": logical,
    }


def enough_fast_chunks(times, n_sets):
    """True when n_sets of the probe times are within 0.6 % of the fastest and the fastest is at
    least 4 % below the slowest: the search of input_arenas_in_fast_memory can stop."""
    ranked = sorted(times)
    return (len(ranked) >= n_sets and ranked[n_sets - 1] <= 1.006 * ranked[0]
            and ranked[0] < 0.96 * ranked[-1])


def choose_chunks(times, n_sets):
    """Indices (ascending) of the chunks that become the input sets: the n_sets fastest, or the
    first n_sets when no probe time stands out by 4 %; None when there are fewer than n_sets."""
    if len(times) < n_sets:
        return None
    if min(times) >= 0.96 * max(times):
        return list(range(n_sets))
    order = sorted(range(len(times)), key=lambda q: (times[q], q))
    return sorted(order[:n_sets])


def input_arenas_in_fast_memory(torch, B, hp, cfg, dev, n_sets):
    """Device memory placement.  Device memory on MI355X comes in parts of about 100 GB (in the
    order a fresh process is handed memory), and the update is 9 % slower when the worker vectors
    lie in the same part as the tables they are added into: with the tables allocated first, the
    same update on the same data takes 13.0 ms on vectors within the first 100 GB and 11.8 ms on
    vectors beyond.  So the input sets are not simply allocated next.  This step allocates chunks
    of the size of one input set one after the other, fills them, and times a probe on each (the
    stride-walk update of the chunk's W vectors into the step's own worker tables: the access
    pattern of the step's update, under a kernel name of its own in a trace; folded workers, which
    have no such tables, the step's own update), until n_sets
    chunks are within 0.6 % of the fastest and at least 4 % faster than the slowest.  Those
    become the input sets; the other chunks are freed.  The search goes on for n_sets + 10 chunks
    (one part alone is 8 chunks of 12.8 GB); when no chunk stands out by then, the first n_sets
    chunks are used.  Returns (arenas, probe times in ms, indices chosen, plain), or
    (None, [], [], None) for inputs too small to place; `plain` are the first n_sets chunks (where
    a fresh process that allocates its inputs right after its tables would have them) when the
    choice fell on others, kept so that the same steps can be timed on them, else None."""
    chunk_bytes = 4 * cfg.d * cfg.W
    if cfg.W < 8 or chunk_bytes < (2 << 30) or not B.cs_bundle_update_launches(hp.params, 8, cfg.d):
        return None, [], [], None
    walk = B.CsParams.from_buffer_copy(hp.params)
    walk.flags |= B.CS_FLAG_NO_VISIT_LIST
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)

    def update(vecs):
        if hp.fold_workers:
            hp.accumulate(vecs)
        else:
            B.cs_sketch_accumulate_bundle(walk, hp.T, vecs)

    def probe(vecs):
        update(vecs)
        e0.record()
        update(vecs)
        e1.record()
        torch.cuda.synchronize()
        return e0.elapsed_time(e1)

    chunks, times = [], []
    for _ in range(n_sets + 10):
        free_bytes, _total = torch.cuda.mem_get_info()
        if free_bytes < chunk_bytes + (8 << 30):
            break
        big = torch.empty(cfg.d * cfg.W, dtype=torch.float32, device=dev)
        big.normal_(0.0, 0.01)
        vecs = [big[w * cfg.d:(w + 1) * cfg.d] for w in range(cfg.W)]
        chunks.append(big)
        times.append(probe(vecs))
        if enough_fast_chunks(times, n_sets):
            break
    chosen = choose_chunks(times, n_sets)
    if chosen is None:
        return None, times, [], None
    arenas = [chunks[q] for q in chosen]
    plain = [chunks[q] for q in range(n_sets)] if chosen != list(range(n_sets)) else None
    del chunks, big, vecs
    torch.cuda.empty_cache()
    return arenas, times, chosen, plain


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--config", type=int, default=4,
                    help="1-5: the benchmark configurations (4 is the headline); 6-8: the sketch "
                         "shapes of the paper's Table 1 (5 x 10^6 / 15 x 180 000 over 90 M, 5 x 180 000 "
                         "over 73 M coordinates; W = 4, k = 100 000, their P), run as --variant top-pk")
    ap.add_argument("--variant", default="sketch-state",
                    choices=["sketch-state", "dense-state", "heavymix", "top-pk", "fused-merge"],
                    help="sketch-state: the headline path (momentum / error feedback as sketches; "
                         "stateless for configs 1-3).  dense-state: Alg. 3 as printed, dense u, v "
                         "per worker.  heavymix: Alg. 1 selection (norm estimate, threshold, random "
                         "fill) on the merged sketch, no state.  top-pk: P = 16 candidates per "
                         "selected coordinate, exact second round, k largest exact sums.  "
                         "fused-merge: sketch-state with the workers summed before they are sketched "
                         "(HotPath(fold_workers=True): no worker tables, no merge pass) -- what a "
                         "device that hosts several workers can do; not the headline path")
    ap.add_argument("--graph", action="store_true",
                    help="also time the same step replayed from a HIP graph (one submission per "
                         "step instead of one per kernel); reported as graph_ms_per_step")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--plain-placement", action="store_true",
                    help="allocate the inputs in the plain order of a fresh process, without "
                         "first looking for the device memory where the update runs fastest")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py: this build runs on ONE GPU only (no collectives, no sharding); "
              "--gpus must be 1", file=sys.stderr)
        sys.exit(2)

    import torch

    import workloads as wl
    from paper_1903_04488_amd import binding as B
    from paper_1903_04488_amd.pipeline import DenseStatePath, HotPath

    if not torch.cuda.is_available():
        print("bench.py: no GPU visible", file=sys.stderr)
        sys.exit(1)
    dev = "cuda:0"
    cfg = wl.ALL_CONFIGS[args.config]
    if cfg.P > 1 and args.variant == "sketch-state":
        args.variant = "top-pk"      # the paper's own shapes come with their P (Table 1 footnotes)
    work = wl.Workload(cfg, dev)
    variant = args.variant
    if variant == "dense-state":
        hp = DenseStatePath(cfg.d, cfg.W, cfg.r, cfg.c, cfg.k, cfg.hash_seed,
                            rho=cfg.rho if cfg.rho is not None else 0.9, device=dev)
    elif variant == "top-pk":
        hp = HotPath(cfg.d, cfg.W, cfg.r, cfg.c, cfg.k, cfg.hash_seed, rho=cfg.rho, device=dev,
                     P=cfg.P if cfg.P > 1 else 16)
    elif variant == "heavymix":
        hp = HotPath(cfg.d, cfg.W, cfg.r, cfg.c, cfg.k, cfg.hash_seed, rho=None, device=dev)
        l2sq = torch.empty(1 + cfg.r, dtype=torch.float64, device=dev)
        n_heavy = torch.empty(1, dtype=torch.int64, device=dev)
    else:
        hp = HotPath(cfg.d, cfg.W, cfg.r, cfg.c, cfg.k, cfg.hash_seed, rho=cfg.rho, device=dev,
                     fold_workers=variant == "fused-merge")

    # inputs resident in HBM before the timed region: a few distinct steps' worth, cycled
    bytes_per_set = 4 * cfg.d * cfg.W
    n_sets = max(1, min(args.steps + args.warmup, int(60e9 // bytes_per_set), 4))
    arenas, probe_ms, chosen, plain_arenas = (
        (None, [], [], None) if args.plain_placement
        else input_arenas_in_fast_memory(torch, B, hp, cfg, dev, n_sets))

    def sets_in(chunks):
        out = [[chunks[t][w * cfg.d:(w + 1) * cfg.d] for w in range(cfg.W)] for t in range(n_sets)]
        for t in range(n_sets):
            for w in range(cfg.W):
                work.gradient(t, w, out=out[t][w])
        return out

    if arenas is None:
        sets = [[work.gradient(t, w) for w in range(cfg.W)] for t in range(n_sets)]
    else:
        sets = sets_in(arenas)
    torch.cuda.synchronize()

    # stage names per variant; stage i runs between events i and i + 1.  The stages of HotPath.step are called as it
    # calls them, but second round and feedback, which begin in one launch there, one by one; where its update goes by way
    # of running sums, merge and momentum come out of the pass that gathers them.  The update itself (all of it, or without the clearing of worker tables where requests add to them) is
    # bracketed by its own pair of events (ev[8], ev[9]) for the roofline figure.
    by_sums = hp._index is not None
    sketch = ["accumulate+merge+momentum", "-", "-"] if by_sums else ["accumulate", "merge+momentum", "-"]
    stages = {"sketch-state": [*sketch, "estimate", "topk", "gather", "feedback"],
              "fused-merge": [*sketch, "estimate", "topk", "gather", "feedback"],
              "top-pk": [*sketch, "estimate", "topk", "gather+select", "feedback"],
              "dense-state": ["dense_momentum", "accumulate", "merge", "estimate", "topk", "gather", "mask"],
              "heavymix": ["accumulate", "merge", "l2sq", "estimate", "heavymix_select", "gather", "-"]}[variant]

    def one_step(g_w, ev=None):
        def mark(i):
            if ev is not None:
                ev[i].record()

        def update(vecs):
            if hp.fold_workers or by_sums:
                mark(8)
                hp.accumulate(vecs)
                mark(9)
                return
            B.cs_bundle_zero(hp.params, hp.T, hp.W)
            mark(8)
            B.cs_sketch_accumulate_bundle(hp.params, hp.T, vecs)
            mark(9)

        mark(0)
        if variant == "dense-state":
            hp.dense_momentum(g_w); mark(1)
            update(hp.v_w); mark(2)
            hp.merge(); mark(3)
            hp.estimate(); mark(4)
            hp.topk(); mark(5)
            hp.gather(hp.v_w); mark(6)
            hp.mask(); mark(7)
        elif variant == "heavymix":
            update(g_w); mark(1)
            hp.merge(); mark(2)
            B.cs_sketch_l2sq(hp.params, hp.S_t, l2sq); mark(3)
            hp.estimate(); mark(4)
            B.cs_heavymix_select(hp.est, cfg.k, l2sq, 12345, hp.cand, hp.est_at_cand, n_heavy,
                                 hp.topk_ws); mark(5)
            hp.gather(g_w); mark(6)
            mark(7)
        else:
            if by_sums:
                mark(8)
                hp.sketch_and_aggregate(g_w)
                mark(9); mark(1); mark(2)
            else:
                update(g_w); mark(1)
                hp.aggregate(); mark(2)
            mark(3)
            hp.estimate(); mark(4)
            hp.topk(); mark(5)
            hp.gather(g_w); mark(6)
            hp.feedback(); mark(7)

    def timed_steps(input_sets):
        """args.warmup untimed steps, then args.steps timed ones; (ms per step, events)"""
        for t in range(args.warmup):
            one_step(input_sets[t % n_sets])
        torch.cuda.synchronize()
        evs = [[torch.cuda.Event(enable_timing=True) for _ in range(10)] for _ in range(args.steps)]
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for t in range(args.steps):
            one_step(input_sets[(args.warmup + t) % n_sets], evs[t])
        torch.cuda.synchronize()
        return (time.perf_counter() - t0) / args.steps * 1e3, evs

    # the same steps on inputs where a fresh process would plainly have them, for the record
    # (state tables are reset in between so that both runs do the same work)
    plain_ms_per_step = None
    if plain_arenas is not None:
        state = [t.clone() for t in (getattr(hp, "S_u", None), getattr(hp, "S_v", None)) if t is not None]
        plain_ms_per_step, _ = timed_steps(sets_in(plain_arenas))
        for t, saved in zip([t for t in (getattr(hp, "S_u", None), getattr(hp, "S_v", None)) if t is not None], state):
            t.copy_(saved)
        del plain_arenas, state
        torch.cuda.empty_cache()

    ms_per_step, events = timed_steps(sets)
    if args.plain_placement or (arenas is not None and plain_ms_per_step is None):
        plain_ms_per_step = ms_per_step          # the inputs are in the plain order
    stage_ms = {}
    for i, name in enumerate(stages):
        stage_ms[name] = sum(ev[i].elapsed_time(ev[i + 1]) for ev in events) / args.steps
    # the update runs as a few launches per group of 8 workers (rows that share a traversal
    # share a launch); the algorithmic bytes of the whole update (every gradient read once,
    # every worker table written once) are spread evenly over those launches
    # (folded workers: one call of several different kernels, taken as a whole; cell lists: one launch; by running sums: a
    # launch per group and 8 rows, with its share of the pass that gathers them)
    n_launch = (1 if hp.fold_workers or hp._cell_lists else (cfg.W + 7) // 8 * ((cfg.r + 7) // 8) if by_sums
                else B.cs_bundle_update_launches(hp.params, cfg.W, cfg.d))
    acc_kernel_ms = sum(ev[8].elapsed_time(ev[9]) for ev in events) / args.steps / n_launch
    per_set = [[] for _ in range(n_sets)]         # the update's time on each resident input set
    for t, ev in enumerate(events):
        per_set[(args.warmup + t) % n_sets].append(ev[8].elapsed_time(ev[9]))
    update_ms_per_set = [round(sum(v) / len(v), 3) if v else None for v in per_set]
    value = cfg.W * cfg.d / (ms_per_step * 1e-3) / 1e9

    tables_written = 1 if variant == "fused-merge" else cfg.W
    alg_bytes = (4.0 * cfg.W * cfg.d + 4.0 * cfg.r * cfg.c * tables_written) / n_launch
    achieved = alg_bytes / (acc_kernel_ms * 1e-3) / 1e9
    step_alg_bytes = (4.0 * cfg.W * cfg.d + 4.0 * cfg.r * cfg.c * tables_written  # update
                      + (0.0 if hp.fold_workers else 4.0 * cfg.r * cfg.c * (cfg.W + 1))   # merge
                      + (4.0 * cfg.r * cfg.c * 5 if cfg.stateful else 0.0)       # momentum
                      + 4.0 * cfg.r * cfg.c + 4.0 * cfg.d                        # estimate
                      + 4.0 * cfg.d                                              # top-k
                      + 4.0 * cfg.k * cfg.W)                                     # gather
    # the streaming-read ceiling of this machine, measured live with the library's plain read kernel:
    # one worker vector read repeatedly, and one whole input set (what a row's pass of the
    # update reads).  Outside the timed steps.
    probe_out = torch.zeros(1, dtype=torch.float32, device=dev)

    def read_rate(vecs, reps):
        B.cs_probe_stream_read(vecs, probe_out)
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(reps):
            B.cs_probe_stream_read(vecs, probe_out)
        e1.record()
        torch.cuda.synchronize()
        return 4.0 * cfg.d * len(vecs) * reps / (e0.elapsed_time(e1) * 1e-3) / 1e9

    stream_one = read_rate(sets[0][:1], 8)
    stream_set = read_rate(sets[0], 3)
    # (measured for the update into worker tables; the fused-merge variant writes one table instead)
    traffic = MEASURED_TRAFFIC_BYTES.get(cfg.cfg) if variant != "fused-merge" and not by_sums else None

    out = {
        "metric": METRIC,
        "value": value,
        "unit": "Gcoords/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_per_step,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic",
        "config": {"workload": f"cfg{cfg.cfg} {cfg.name}", "variant": variant, "d": cfg.d,
                   "W": cfg.W, "r": cfg.r, "c": cfg.c, "k": cfg.k, "rho": cfg.rho,
                   "P": getattr(hp, "P", 1),
                   "input_sets_resident": n_sets},
        "pct_hbm_peak_whole_step": 100.0 * step_alg_bytes / (ms_per_step * 1e-3) / 1e9 / HBM_PEAK_GBS,
        "pct_stream_read_whole_step": 100.0 * step_alg_bytes / (ms_per_step * 1e-3) / 1e9 / stream_set,
        "stream_read": {"one_vector_GBs": stream_one, "one_input_set_GBs": stream_set,
                        "kernel": "cs_probe_stream_read (plain 16-byte loads)"},
        "placement": {"probe": ("the step's" if hp.fold_workers else "stride-walk")
                      + " update of successive chunks of one input set's size",
                      "probe_ms": [round(t, 3) for t in probe_ms],
                      "chunks_used_for_inputs": chosen,
                      "update_ms_per_input_set": update_ms_per_set,
                      "plain_ms_per_step": plain_ms_per_step,
                      "plain_value": (cfg.W * cfg.d / (plain_ms_per_step * 1e-3) / 1e9
                                      if plain_ms_per_step else None),
                      "note": "plain_*: the same timed steps with the inputs allocated in the plain "
                              "order of a fresh process (the first chunks), before the headline run"},
        "stage_ms": stage_ms,
        "stage_Gcoords_s": {name: (cfg.W if name.startswith(("accumulate", "dense_momentum")) else 1) * cfg.d
                            / (stage_ms[name] * 1e-3) / 1e9
                            for name in ("accumulate", "accumulate+merge+momentum", "dense_momentum", "estimate",
                                         "topk", "heavymix_select")
                            if stage_ms.get(name)},
        "roofline": {
            "kernel": ("cs_vectors_sum and the sketch of the sum" if variant == "fused-merge"
                       else "cs_bundle_sketch (k_accumulate_visits into running sums, k_gather_sums)" if by_sums
                       else "k_accumulate_visits (all launches of cs_sketch_accumulate_bundle)"),
            "bound": "hbm",
            "achieved": achieved,
            "peak": HBM_PEAK_GBS,
            "unit": "GB/s",
            "frac": achieved / HBM_PEAK_GBS,
            "traffic": traffic,
            "traffic_GBs": traffic / (acc_kernel_ms * 1e-3) / 1e9 if traffic else None,
            "avg_launch_ms": acc_kernel_ms,
            "launches_per_step": n_launch,
            "algorithmic_bytes_per_launch": alg_bytes,
        },
    }
    if args.graph:
        from paper_1903_04488_amd.pipeline import GraphedStep
        graphed = GraphedStep(hp, sets[0])
        for _ in range(args.warmup):
            graphed.replay()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(args.steps):
            graphed.replay()
        torch.cuda.synchronize()
        out["graph_ms_per_step"] = (time.perf_counter() - t0) / args.steps * 1e3
    if not args.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline(cfg, work)
    print(json.dumps(out))


if __name__ == "__main__":
    main()
