#!/usr/bin/env python3
"""Benchmark: MPDP exact join ordering on the 25-relation star (one GPU).

A step optimizes a batch of 16 seeded 25-relation star queries (hub 0 plus
24 leaves, card 10^U(2,8), sel U(0.1,1)/max card, C_out in binary64) end to
end through the C-ABI (mpdp_optimize_ws): query upload, every DP level on
the GPU, plan readback.  The query inputs are host arrays of a few hundred
bytes; the memo lives in HBM.

value      csg-cmp pairs (unordered) per second over the timed steps
           (#ccp = 24 * 2^23 = 201,326,592 per query, fixed by the graph)
roofline   the dominant kernel's algorithmic bytes over its HIP-event time
cpu_baseline  the CPU oracle (MPDP in plain C, one thread) on one query

Besides the headline (timed region: the star-25 steps only), the same JSON
line carries two untimed reports:
batch      4096 mixed queries of 8-20 relations in one persistent launch:
           kernel time, per-query latency p50/p99 (device clock from the
           launch start), queries/s; then the per-query schedules chosen by
           the library's autotuner and the batch replayed as one captured HIP
           graph with them (graph_tuned)
large      100-1000 relations (snowflake, depth 4, random cross edges):
           GOO, IDP2 (k 15, 25), UnionDP (k 15) and the learned UnionDP
           (k 15, scorer trained on the GPU first): plan cost normalized to
           the best plan found per query, and optimization time; the learned
           vs plain UnionDP cost ratio; and on held-out 20-26 relation
           queries both UnionDPs' ratio to the exact optimum
configs    the paper-shaped single queries: star 12, snowflake 25 (both
           models), cycle of 20-30 relations plus 5-15 chords, clique 18:
           optimize time median / p99 over the seeds, ccp pairs per second
ablations  the same optimizer with DPSUB's vertex-based candidates on the GPU,
           the tree kernel without its LDS compaction, and with prune not
           fused into evaluate (results unchanged)
cpu_allcores  the library's multi-threaded CPU MPDP on the star, on one
           GPU's share of the host's cores (16 threads at most; the host's
           core count and CPU model are recorded), next to the single-thread
           oracle of cpu_baseline
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import statistics
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "ccp pairs evaluated/sec + optimize time (ms) 25-rel star; learned vs plain cost ratio"
HBM_PEAK_GBS = 8000.0
CPU_SHARE_PER_GPU = 16   # host threads one GPU's jobs may use on a shared GPU host
TRAFFIC_FILE = os.path.join(ROOT, "profiles", "traffic_level_tree_star25.json")
KERNEL_SRCS = [os.path.join(ROOT, "paper_2202_13511_amd", "csrc", f)
               for f in ("mpdp_kernels.hip", "mpdp_device.h", "mpdp_internal.h")]

# Algorithmic bytes (per the memo layout: cost f64, card f64, left u32, op u8):
#   per csg-cmp pair, C_out gathers the cost of the non-singleton side: 8 B
#   per connected set, one memo entry is written: 21 B
PAIR_BYTES_COUT = 8
PAIR_BYTES_PGLIKE = 16
SET_BYTES = 21


def kernel_hash() -> str:
    h = hashlib.sha256()
    for f in KERNEL_SRCS:
        h.update(open(f, "rb").read())
    return h.hexdigest()[:16]


def load_traffic():
    try:
        t = json.load(open(TRAFFIC_FILE))
    except (OSError, ValueError):
        return None
    if t.get("kernel_source_sha256_16") != kernel_hash():
        return None
    return t.get("traffic_bytes_per_launch")


def main() -> int:
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--queries", type=int, default=16)
    ap.add_argument("--n", type=int, default=25)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-pglike", action="store_true")
    ap.add_argument("--copy-probe-mib", type=int, default=0,
                    help="also run a plain device copy of this size (counter scaling)")
    ap.add_argument("--no-batch", action="store_true")
    ap.add_argument("--no-large", action="store_true")
    ap.add_argument("--no-ablations", action="store_true")
    ap.add_argument("--no-configs", action="store_true")
    ap.add_argument("--profile", choices=sorted(PROFILE_WORKLOADS),
                    help="only run this workload a few times (a short program for rocprofv3) and print one line")
    ap.add_argument("--profile-cost-model", type=int, default=0)
    ap.add_argument("--profile-reps", type=int, default=2)
    args = ap.parse_args()

    if args.gpus != 1:
        print(f"bench.py runs on exactly one GPU; --gpus {args.gpus} is not supported "
              f"(the optimizer is a single-GPU program)", file=sys.stderr)
        return 2

    import numpy as np
    import torch

    from paper_2202_13511_amd import mpdp, workloads

    mpdp.load()  # fails loudly without the HIP library
    if not torch.cuda.is_available():
        print("bench.py needs a GPU", file=sys.stderr)
        return 1
    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    if args.profile:
        return profile_workload(mpdp, workloads, dev, args.profile, args.profile_cost_model, args.profile_reps,
                                args.copy_probe_mib)
    n = args.n
    queries = [workloads.star(n, s) for s in range(args.queries)]
    ccp_per_query = (n - 1) * 2 ** (n - 2)

    def run_batch(cm, ws, per_query_ms, kern, flags):
        total_ccp = 0
        for q in queries:
            t = time.perf_counter()
            r = mpdp.mpdp_optimize_ws(q, cm, ws, flags=flags)
            per_query_ms.append((time.perf_counter() - t) * 1e3)
            kern["eval_ms"] += r.stats["ms_eval"]
            kern["filter_ms"] += r.stats["ms_filter"]
            kern["eval_launches"] += r.stats["eval_launches"]
            kern["sets"] += r.stats["connected_sets"]
            kern["pairs"] += r.stats["ccp_pairs"]
            if r.stats["ccp_pairs"] != ccp_per_query:
                raise RuntimeError(f"{q.name}: {r.stats['ccp_pairs']} ccp, expected {ccp_per_query}")
            total_ccp += r.stats["ccp_pairs"]
        return total_ccp

    def timed(cm, steps, warmup, flags=0):
        ws = mpdp.workspace(n, cm, dev)
        for _ in range(warmup):
            run_batch(cm, ws, [], dict(eval_ms=0.0, filter_ms=0.0, eval_launches=0, sets=0, pairs=0), flags)
        per_query = []
        kern = dict(eval_ms=0.0, filter_ms=0.0, eval_launches=0, sets=0, pairs=0)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        ccp = 0
        for _ in range(steps):
            ccp += run_batch(cm, ws, per_query, kern, flags)
        torch.cuda.synchronize()
        dt = time.perf_counter() - t0
        del ws
        torch.cuda.empty_cache()
        return ccp, dt, per_query, kern

    # pass 1: throughput and optimize time, no per-kernel events in the stream
    ccp, dt, per_query, _ = timed(mpdp.MPDP_COST_COUT, args.steps, args.warmup)
    value = ccp / dt
    # pass 2: the same steps with HIP events around every level kernel, recorded
    # by the library on the stream it launches on (the events add gaps between
    # kernels, not kernel time, so they are kept out of pass 1)
    _, dt_ev, _, kern = timed(mpdp.MPDP_COST_COUT, args.steps, 1, mpdp.MPDP_FLAG_TIMING)
    per_query.sort()
    p50 = statistics.median(per_query)
    p99 = per_query[min(len(per_query) - 1, int(round(0.99 * (len(per_query) - 1))))]

    # roofline of the dominant kernel (the evaluate kernel), from HIP events.
    # A tree query has no filter kernel, so its "filter" interval is an empty
    # pair of events recorded just before each level kernel: what a pair of
    # markers costs on this stream.  The kernel's own duration is the event
    # interval around it less that cost (the trace's kernel time agrees).
    launches = max(kern["eval_launches"], 1)
    alg_bytes = kern["pairs"] * PAIR_BYTES_COUT + kern["sets"] * SET_BYTES
    marker_ms = kern["filter_ms"]
    eval_s = max(kern["eval_ms"] - marker_ms, 0.0) / 1e3
    achieved = alg_bytes / eval_s / 1e9 if eval_s > 0 else 0.0
    traffic = load_traffic()

    out = {
        "metric": METRIC,
        "value": value,
        "unit": "ccp pairs/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": dt / args.steps * 1e3,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64",
        "data": "synthetic",
        "config": {
            "workload": f"star{n}: hub 0 + {n - 1} leaves, card 10^U(2,8), sel U(0.1,1)/max(card), "
                        f"seeds 0..{args.queries - 1}, C_out, exact bushy DP",
            "queries_per_step": args.queries,
            "relations": n,
            "cost_model": "C_out",
            "ccp_per_query": ccp_per_query,
        },
        "optimize_ms_p50": p50,
        "optimize_ms_p99": p99,
        "kernel_ms_per_query": {
            "eval": kern["eval_ms"] / len(per_query),
            "filter": kern["filter_ms"] / len(per_query),
        },
        "ms_per_step_with_events": dt_ev / args.steps * 1e3,
        "roofline": {
            "kernel": "k_level_flat + k_level_tree_split <C_out>",
            "bound": "hbm",
            "achieved": achieved,
            "peak": HBM_PEAK_GBS,
            "unit": "GB/s",
            "frac": achieved / HBM_PEAK_GBS,
            "traffic": traffic,
            "algorithmic_bytes_per_launch": alg_bytes / launches,
            "avg_launch_ms": eval_s * 1e3 / launches,
            "avg_event_interval_ms": kern["eval_ms"] / launches,
            "marker_ms_per_launch": marker_ms / launches,
        },
    }

    if not args.no_pglike:
        ccp2, dt2, pq2, _ = timed(mpdp.MPDP_COST_PGLIKE, max(1, args.steps // 5), 1)
        _, _, _, k2 = timed(mpdp.MPDP_COST_PGLIKE, max(1, args.steps // 5), 0, mpdp.MPDP_FLAG_TIMING)
        pq2.sort()
        out["pglike"] = {
            "value": ccp2 / dt2,
            "optimize_ms_p50": statistics.median(pq2),
            "eval_ms_per_query": (k2["eval_ms"] - k2["filter_ms"]) / len(pq2),
            "eval_achieved_GBs": (k2["pairs"] * PAIR_BYTES_PGLIKE + k2["sets"] * SET_BYTES)
                                 / ((k2["eval_ms"] - k2["filter_ms"]) / 1e3) / 1e9
                                 if k2["eval_ms"] > k2["filter_ms"] else None,
        }

    if args.copy_probe_mib:
        nb = args.copy_probe_mib << 20
        a = torch.ones(nb, dtype=torch.uint8, device=dev)
        b = torch.empty_like(a)
        torch.cuda.synchronize()
        b.copy_(a)
        torch.cuda.synchronize()
        out["copy_probe_bytes"] = nb

    if not args.no_batch:
        out["batch"] = bench_batch(mpdp, workloads, np)

    if not args.no_configs:
        out["configs"] = bench_configs(mpdp, workloads, np, dev)
    if not args.no_large:
        out["large"] = bench_large(mpdp, workloads, np)

    if not args.no_ablations:
        out["ablations"] = bench_ablations(mpdp, workloads, dev)
        host = host_cpu()
        threads = host["cpu_share"]
        q = queries[0]
        t = time.perf_counter()
        r = mpdp.mpdp_optimize_cpu(q, mpdp.MPDP_COST_COUT, threads)
        cdt = time.perf_counter() - t
        cpu_rate = r.stats["ccp_pairs"] / cdt
        out["cpu_allcores"] = {"value": cpu_rate, "unit": "ccp pairs/s", "threads": threads,
                               "optimize_ms": cdt * 1e3, "query": q.name, "gpu_speedup": value / cpu_rate,
                               **host}

    if not args.no_cpu_baseline:
        import oracle
        q = queries[0]
        t = time.perf_counter()
        m = oracle.mpdp(q, oracle.COST_COUT)
        cdt = time.perf_counter() - t
        gpu_root = mpdp.mpdp_optimize(q, mpdp.MPDP_COST_COUT).cost
        out["cpu_baseline"] = {
            "value": (m.ccp_ordered // 2) / cdt,
            "unit": "ccp pairs/s",
            "cores": 1,
            "kind": "oracle",
            "sample": f"{q.name}: one query of the batch, C_out, oracle MPDP (plain C, one thread), "
                      f"{cdt:.1f} s",
            "optimize_ms": cdt * 1e3,
            "cpu_model": host_cpu()["cpu_model"],
            "root_cost_bits_equal": bool(np.float64(gpu_root).view(np.uint64)
                                         == np.float64(m.root_cost).view(np.uint64)),
        }

    print(json.dumps(out), flush=True)
    return 0


def host_cpu():
    """The host's CPU model and core counts.  A GPU host shared by several
    GPUs gives each one a share of its cores (CPU_SHARE_PER_GPU threads):
    the all-cores baseline uses that share, or every core the process may
    run on if fewer."""
    model = ""
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    model = line.split(":", 1)[1].strip()
                    break
    except OSError:
        pass
    visible = os.cpu_count() or 1
    allowed = len(os.sched_getaffinity(0)) if hasattr(os, "sched_getaffinity") else visible
    return {"cpu_model": model, "host_cores": visible, "cores_allowed": allowed,
            "cpu_share": max(1, min(allowed, CPU_SHARE_PER_GPU))}


# Short programs for the profiler: one family of kernels each.
PROFILE_WORKLOADS = {
    "star25": "star 25, seeds 0-1 (tree level kernels)",
    "snowflake25": "snowflake 25, seeds 0-3 (tree level kernels, sparse levels)",
    "cycle_p99": "cycle30+12-s15, the slowest C3a seed (pair search kernels)",
    "cycle_median": "cycle27+8-s8, a median C3a seed",
    "clique18": "clique 18, seed 0 (bitmap kernels)",
    "batch": "the 4096-query mixed batch, one persistent launch",
}


def profile_workload(mpdp, workloads, dev, name, cm, reps, copy_mib):
    import torch
    if name == "batch":
        qs = workloads.batch_mixed(4096, 0)
        ws = mpdp.batch_workspace(qs)
        for _ in range(reps):
            r = mpdp.mpdp_optimize_batch(qs, cm, ws, flags=mpdp.MPDP_FLAG_TIMING)
        info = {"queries": len(qs), "kernel_ms": r.stats["ms_kernel"], "ccp": r.stats["ccp_pairs"]}
    else:
        qs = {"star25": [workloads.star(25, s) for s in range(2)],
              "snowflake25": [workloads.snowflake(25, s) for s in range(4)],
              "cycle_p99": [workloads.cycle_chords(15)],
              "cycle_median": [workloads.cycle_chords(8)],
              "clique18": [workloads.clique(18, 0)]}[name]
        ws = mpdp.workspace(max(q.n for q in qs), cm, dev)
        info = {"queries": [q.name for q in qs], "ms": [], "ccp": 0, "evaluated": 0, "sets": 0}
        for _ in range(reps):
            for q in qs:
                t = time.perf_counter()
                r = mpdp.mpdp_optimize_ws(q, cm, ws)
                info["ms"].append((time.perf_counter() - t) * 1e3)
        for q in qs:
            r = mpdp.mpdp_optimize_ws(q, cm, ws)
            info["ccp"] += r.stats["ccp_pairs"]
            info["evaluated"] += r.stats["evaluated_pairs"]
            info["sets"] += r.stats["connected_sets"]
    if copy_mib:
        nb = copy_mib << 20
        a = torch.ones(nb, dtype=torch.uint8, device=dev)
        b = torch.empty_like(a)
        torch.cuda.synchronize()
        b.copy_(a)
        torch.cuda.synchronize()
        info["copy_probe_bytes"] = nb
    torch.cuda.synchronize()
    print(json.dumps({"profile": name, "cost_model": cm, "reps": reps, **info}), flush=True)
    return 0


def bench_batch(mpdp, workloads, np, count=4096, runs=3):
    """Config 4: one persistent launch over `count` mixed queries."""
    import torch
    qs = workloads.batch_mixed(count, 0)
    ws = mpdp.batch_workspace(qs)
    out = {}
    for cm, name in ((mpdp.MPDP_COST_COUT, "C_out"), (mpdp.MPDP_COST_PGLIKE, "PG-like")):
        mpdp.mpdp_optimize_batch(qs, cm, ws, flags=mpdp.MPDP_FLAG_TIMING)  # warm-up
        best = None
        for _ in range(runs):
            t = time.perf_counter()
            r = mpdp.mpdp_optimize_batch(qs, cm, ws, flags=mpdp.MPDP_FLAG_TIMING)
            wall = (time.perf_counter() - t) * 1e3
            if best is None or r.stats["ms_kernel"] < best[0].stats["ms_kernel"]:
                best = (r, wall)
        r, wall = best
        lat = np.sort(r.latency_us)
        out[name] = {
            "kernel_ms": r.stats["ms_kernel"],
            "call_ms": wall,
            "queries_per_s": count / (r.stats["ms_kernel"] / 1e3),
            "latency_us_p50": float(lat[len(lat) // 2]),
            "latency_us_p99": float(lat[int(0.99 * (len(lat) - 1))]),
            "latency_us_max": float(lat[-1]),
            "ccp_pairs_per_s": r.stats["ccp_pairs"] / (r.stats["ms_kernel"] / 1e3),
        }
        # per-query schedules from the autotuner (untimed), then the batch as
        # one captured HIP graph replayed with those schedules
        t = time.perf_counter()
        sched, tst = mpdp.mpdp_batch_autotune(qs, cm, ws, reps=2)
        tune_s = time.perf_counter() - t
        g = mpdp.BatchGraph(qs, cm, ws)
        try:
            g.run(qs, schedules=sched)  # warm-up
            gbest = None
            for _ in range(runs):
                t = time.perf_counter()
                gr = g.run(qs, schedules=sched)
                gwall = (time.perf_counter() - t) * 1e3
                if gbest is None or gwall < gbest[1]:
                    gbest = (gr, gwall)
        finally:
            g.close()
        gr, gwall = gbest
        assert gr.costs == r.costs  # schedules and replay leave every result unchanged
        glat = np.sort(gr.latency_us)
        picked = {}
        for tc, hc in sched:
            picked[f"{tc}/{hc}"] = picked.get(f"{tc}/{hc}", 0) + 1
        out[name]["graph_tuned"] = {
            "call_ms": gwall,
            "span_ms": float(glat[-1]) / 1e3,
            "queries_per_s": count / (float(glat[-1]) / 1e6),  # device span, as kernel_ms above
            "queries_per_s_call": count / (gwall / 1e3),        # host call, packing and unpacking included
            "latency_us_p50": float(glat[len(glat) // 2]),
            "latency_us_p99": float(glat[int(0.99 * (len(glat) - 1))]),
            "latency_us_max": float(glat[-1]),
            "tuning_s": tune_s, "tune_classes": tst["classes"], "tune_launches": tst["launches"],
            "est_default_ms": tst["est_default_ms"], "est_tuned_ms": tst["est_tuned_ms"],
            "schedules_tree_chunk_over_heavy_chunks": picked,
        }
    del ws
    torch.cuda.empty_cache()
    return {"workload": f"{count} queries, n ~ U{{8..20}}, chain/star/cycle/snowflake/random mix, seed 0",
            "workgroups": 512, "runs": runs, **out}


def bench_configs(mpdp, workloads, np, dev):
    """The paper-shaped single-query workloads (untimed by the headline):
    end-to-end optimize time per query (best of `reps` after a warm-up),
    median and p99 over the seeds, and ccp pairs per second over all of
    them.  C3a runs each seed once: its larger queries take up to a second."""
    import torch
    specs = [("C1 star12", lambda s: workloads.star(12, s), 64, (mpdp.MPDP_COST_COUT,), 3),
             ("C2 snowflake25", lambda s: workloads.snowflake(25, s), 64,
              (mpdp.MPDP_COST_COUT, mpdp.MPDP_COST_PGLIKE), 2),
             ("C3a cycle20-30+5-15 chords", lambda s: workloads.cycle_chords(s), 32, (mpdp.MPDP_COST_COUT,), 0),
             ("C3b clique18", lambda s: workloads.clique(18, s), 32,
              (mpdp.MPDP_COST_COUT, mpdp.MPDP_COST_PGLIKE), 1)]
    out = {}
    for name, gen, seeds, cms, reps in specs:
        qs = [gen(s) for s in range(seeds)]
        for cm in cms:
            ws = mpdp.workspace(max(q.n for q in qs), cm, dev)
            mpdp.mpdp_optimize_ws(qs[0], cm, ws)  # warm-up
            ms, ccp = [], 0
            for q in qs:
                best = None
                for _ in range(max(reps, 1)):
                    t = time.perf_counter()
                    r = mpdp.mpdp_optimize_ws(q, cm, ws)
                    dt = (time.perf_counter() - t) * 1e3
                    best = dt if best is None else min(best, dt)
                ms.append(best)
                ccp += r.stats["ccp_pairs"]
            del ws
            torch.cuda.empty_cache()
            ms_s = sorted(ms)
            out[f"{name} {'C_out' if cm == mpdp.MPDP_COST_COUT else 'PG-like'}"] = {
                "queries": seeds, "optimize_ms_median": float(ms_s[len(ms_s) // 2]),
                "optimize_ms_p99": float(ms_s[min(len(ms_s) - 1, int(round(0.99 * (len(ms_s) - 1))))]),
                "optimize_ms_max": float(ms_s[-1]), "ccp_pairs_per_s": ccp / (sum(ms) / 1e3)}
    return out


def bench_ablations(mpdp, workloads, dev, reps=5):
    """Optimize time (min of reps) with and without the enhancements."""
    import torch

    def best_ms(q, flags):
        ws = mpdp.workspace(q.n, mpdp.MPDP_COST_COUT, dev)
        mpdp.mpdp_optimize_ws(q, mpdp.MPDP_COST_COUT, ws, flags=flags)
        ts, st = [], None
        for _ in range(reps):
            t = time.perf_counter()
            r = mpdp.mpdp_optimize_ws(q, mpdp.MPDP_COST_COUT, ws, flags=flags)
            ts.append((time.perf_counter() - t) * 1e3)
            st = r.stats
        del ws
        torch.cuda.empty_cache()
        return min(ts), st

    out = {"no_compaction": {}, "unfused_prune": {}, "dpsub": {}}
    for q in (workloads.star(25, 0), workloads.snowflake(25, 0)):
        a, _ = best_ms(q, 0)
        b, _ = best_ms(q, mpdp.MPDP_FLAG_ABLATE_NO_COMPACTION)
        out["no_compaction"][q.name] = {"mpdp_ms": a, "ablated_ms": b, "slowdown": b / a}
        b, _ = best_ms(q, mpdp.MPDP_FLAG_ABLATE_UNFUSED_PRUNE)
        out["unfused_prune"][q.name] = {"mpdp_ms": a, "ablated_ms": b, "slowdown": b / a}
    for q in (workloads.star(20, 0), workloads.snowflake(20, 1), workloads.clique(14, 0)):
        a, sa = best_ms(q, 0)
        b, sb = best_ms(q, mpdp.MPDP_FLAG_ABLATE_DPSUB)
        out["dpsub"][q.name] = {"mpdp_ms": a, "dpsub_ms": b, "slowdown": b / a,
                                "mpdp_candidates": sa["evaluated_pairs"], "dpsub_candidates": sb["evaluated_pairs"]}
    return out


def bench_large(mpdp, workloads, np):
    """Config 5: heuristics on 100-1000 relations; learned vs plain UnionDP."""
    from paper_2202_13511_amd import scorer
    M = mpdp
    methods = [("goo", M.MPDP_LARGE_GOO, 2), ("idp2_15", M.MPDP_LARGE_IDP2, 15), ("idp2_25", M.MPDP_LARGE_IDP2, 25),
               ("uniondp_15", M.MPDP_LARGE_UNIONDP, 15), ("uniondp_20", M.MPDP_LARGE_UNIONDP, 20),
               ("uniondp_25", M.MPDP_LARGE_UNIONDP, 25), ("learned_uniondp_15", M.MPDP_LARGE_UNIONDP_LEARNED, 15),
               ("learned_uniondp_25", M.MPDP_LARGE_UNIONDP_LEARNED, 25)]
    plain_uniondp = ("uniondp_15", "uniondp_20", "uniondp_25")
    res = {"workload": "large_snowflake(n, seed): depth <= 4, round(n/20) cross edges; n in {100, 300, 1000}, "
                       "seeds 0..2; costs normalized to the best plan found per query",
           "train": {}, "cost_models": {}}
    for cm, cname in ((M.MPDP_COST_COUT, "C_out"), (M.MPDP_COST_PGLIKE, "PG-like")):
        t = time.perf_counter()
        block, log = scorer.train(cm, seed=1, queries=300, rounds=4, steps=3000)
        res["train"][cname] = {"seconds": time.perf_counter() - t, "examples": log.examples[-1],
                               "final_loss": log.loss[-1]}
        per_n = {}
        ratios_lp = []
        ratios_eq = []  # learned (k 15 or 25) vs the best plain UnionDP run that took no longer
        ratios_lp25 = []
        for n in (100, 300, 1000):
            rows = {name: [] for name, _, _ in methods}
            times = {name: [] for name, _, _ in methods}
            for seed in range(3):
                q = workloads.large_snowflake(n, seed)
                costs = {}
                for name, meth, k in methods:
                    t = time.perf_counter()
                    r = M.mpdp_optimize_large(q, cm, meth, k, scorer=block if "learned" in name else None)
                    times[name].append((time.perf_counter() - t) * 1e3)
                    costs[name] = r.cost
                best = min(costs.values())
                for name in costs:
                    rows[name].append(costs[name] / best)
                ratios_lp.append(costs["learned_uniondp_15"] / costs["uniondp_15"])
                ratios_lp25.append(costs["learned_uniondp_25"] / costs["uniondp_25"])
                for ln, pk in (("learned_uniondp_15", "uniondp_15"), ("learned_uniondp_25", "uniondp_25")):
                    t_l = times[ln][-1]
                    eq = [costs[nm] for nm in plain_uniondp if times[nm][-1] <= t_l] or [costs[pk]]
                    ratios_eq.append(costs[ln] / min(eq))
            per_n[str(n)] = {name: {"cost_ratio_mean": float(np.mean(rows[name])),
                                    "ms_mean": float(np.mean(times[name]))} for name in rows}
        held = scorer.training_queries(40, 99)
        plain, learned = scorer.compare_small(block, cm, held, 15)
        res["cost_models"][cname] = {
            "by_n": per_n,
            "learned_vs_plain_uniondp_geomean": float(np.exp(np.mean(np.log(ratios_lp)))),
            "learned_vs_plain_uniondp_k25_geomean": float(np.exp(np.mean(np.log(ratios_lp25)))),
            "learned_vs_plain_uniondp_equal_time_geomean": float(np.exp(np.mean(np.log(ratios_eq)))),
            "small_vs_exact_geomean": {"uniondp_15": float(np.exp(np.mean(np.log(plain)))),
                                       "learned_uniondp_15": float(np.exp(np.mean(np.log(learned))))},
        }
    return res


if __name__ == "__main__":
    sys.exit(main())
