"""Benchmark: balanced butterfly counting on one MI355X.

One step is one full bbc_count call on a graph already resident in HBM:
input checks, degrees, vertex-priority ranks, degree-ordered CSR, schedule,
wedge aggregation and the 8-byte result.  The workload is the Chung-Lu
power-law graph with |U| = 1,000,000, |V| = 500,000 and 20M edges (gamma 2.1
on both sides, largest expected degree 50,000, P(-) = 0.2), seed 1.

Prints one JSON line.  value = wedges/s, where the wedges are
sum over centres c of C(deg c, 2): every wedge u - c - w with w ranked above
u (the count from both sides covers them by walking fewer, so value is not a
rate of wedges walked there: wedges_walked and kernel_wedges_walked_per_s, and
the roofline, use the wedges it does walk).  The line also carries the batched measurement
(graphs/s of 10,000 graphs of uneven size, one captured batch plan, against
a loop of plain per-graph calls), the six sign-pattern classes on the same
graph, balanced (2,k)-bicliques for k = 2..4 on it, batches of 1,000 and
100,000 edge updates on it (the change of the count against a full
recount), the
dense-block
workload (hybrid int8 matrix-core path against the sparse-only path), the
roofline of the wedge kernel and the CPU oracle's rate.

The main graph's configuration (kernel shape, grid, schedule, queue chunk,
wave-regime threshold) is chosen by the library's autotuner on that graph
before the timed steps (untimed, like the batch plan's); the time with the
library's defaults is reported beside it (--no-tune skips the tuning).
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

WORKLOAD = "powerlaw-1m-500k-20m"
HYBRID_WORKLOAD = "hybrid-2m-1m-50m-16x4096"
HBM_PEAK_GBS = 8000.0  # MI355X HBM3E, 8 TB/s
INT8_PEAK_TOPS = 5000.0  # MI355X dense int8 matrix throughput, 5.0 POPS

# HBM traffic of one call's walk launches (three regimes) on the default
# workload with the library's defaults, from two rocprofv3 --pmc runs
# (FETCH_SIZE, then WRITE_SIZE, KiB per dispatch), each scaled by what the
# counter reads for a 1 GiB device copy (fetch x 2.000, write x 1.000).
# Valid only for the kernel sources it was taken on: the bench reports null
# once their hash differs.
KERNEL_SOURCES = ["paper_2601_17707_amd/csrc/" + f for f in ("top_walk.hip", "top.h", "band.h", "bbc_internal.h")]
MEASURED_TRAFFIC = dict(kernel="k_top_bands + k_top_hash + k_top_light", workload=WORKLOAD, bytes=27826566368,
                        sources_sha256="e7df91d8f2e7ee63d0d356119757118afee38d80aaef9fef632e293386f36e5f",
                        summary="profiles/k_top_powerlaw-1m-500k-20m_pmc.md")


def measured_traffic(workload: str):
    """The recorded traffic if it was taken on this workload and on the
    kernel sources as they are now, else None."""
    import hashlib

    if workload != MEASURED_TRAFFIC["workload"]:
        return None
    h = hashlib.sha256()
    for f in KERNEL_SOURCES:
        with open(os.path.join(ROOT, f), "rb") as fh:
            h.update(fh.read())
    return MEASURED_TRAFFIC["bytes"] if h.hexdigest() == MEASURED_TRAFFIC["sources_sha256"] else None


def two_sided_wedges(g) -> int:
    """Wedges that the count from both sides walks: x - y - w with y and w
    below x in the order (degree class, side with U below V, id), the classes
    exact below 16 and of three mantissa bits above.  A list y of d entries
    with p of them not above y gives C(d, 2) - C(p, 2)."""
    import numpy as np

    def classes(d):
        e = np.maximum(np.frexp(np.maximum(d, 1).astype(np.float64))[1] - 1, 4)
        return np.where(d < 16, d, 16 + (e - 4) * 8 + ((d >> (e - 3)) & 7))

    d_u = np.diff(g.offsets).astype(np.int64)
    adj = np.asarray(g.adj)
    d_v = np.bincount(adj, minlength=g.n_v).astype(np.int64)
    u = np.repeat(np.arange(g.n_u), d_u)
    v_above = classes(d_v)[adj] >= classes(d_u)[u]
    p_u = d_u - np.bincount(u[v_above], minlength=g.n_u)
    p_v = d_v - np.bincount(adj[~v_above], minlength=g.n_v)
    return int(sum(((d * (d - 1) - p * (p - 1)) // 2).sum() for d, p in ((d_u, p_u), (d_v, p_v))))


def two_sided_bytes(g, walked: int) -> int:
    """Bytes the two-sided walk must move: one 4-byte list entry per wedge it
    walks, 16 bytes per middle (entry, end of its wedges, list start, index
    row; every edge is one) and 12 per vertex (schedule entry, list range)."""
    return 4 * walked + 16 * int(g.m) + 12 * (g.n_u + g.n_v)


def algorithmic_bytes(stats: dict) -> int:
    """Bytes the one-sided wedge kernel must move: one 4-byte centre-list entry per
    wedge, 13 bytes per anchor edge (centre id 4, sign 1, list position 4,
    centre-list end 4) and 12 per anchor (schedule entry 4, two offsets)."""
    return 4 * int(stats["wedges"]) + 13 * int(stats["n_edges"]) + 12 * int(stats["n_anchor"])


def cpu_baseline(g, wedges: int, budget_s: float = 15.0) -> dict:
    """The serial oracle (Algorithm 1) timed on this host on a bounded sample
    of the same graph: the anchors with the lowest ids (ids are a random
    permutation, so this is a random anchor sample).  The oracle's own
    transpose is timed separately (an empty anchor range) and left out of the
    rate, which is wedges bucketed per second of counting on one core."""
    import oracle

    def timed(lo, hi):
        t0 = time.perf_counter()
        part, w = oracle.count_anchors(g, lo, hi)
        return time.perf_counter() - t0, w

    n_s = g.n_u if g.n_u < g.n_v else g.n_v
    t_setup, _ = timed(0, 0)
    pilot = max(1, n_s // 500)
    t1, w1 = timed(0, pilot)
    rate = w1 / max(t1 - t_setup, 1e-6)
    k = int(min(n_s, max(pilot, n_s * budget_s * rate / max(wedges, 1))))
    t2, w2 = timed(0, k)
    dt = max(t2 - t_setup, 1e-9)
    h = host_info()
    return dict(value=w2 / dt / 1e9, unit="G/s", cores=1, host_cores=h["cores"], host_model=h["model"], kind="oracle",
                sample=f"anchors 0..{k - 1} of {n_s} ({w2} wedges, {100.0 * w2 / max(wedges, 1):.2f}% of the "
                       f"graph) counted in {dt:.1f} s; oracle transpose {t_setup:.1f} s excluded",
                full_graph_estimate_s=wedges / (w2 / dt) + t_setup)


def host_info() -> dict:
    """Host cores (as this process sees them) and the CPU model."""
    model = ""
    try:
        with open("/proc/cpuinfo") as f:
            for ln in f:
                if ln.startswith("model name"):
                    model = ln.split(":", 1)[1].strip()
                    break
    except OSError:
        pass
    n = len(os.sched_getaffinity(0)) if hasattr(os, "sched_getaffinity") else os.cpu_count()
    return dict(cores=n, logical_cpus=os.cpu_count(), model=model)


def cpu_multicore(g, wedges: int, total: int) -> dict:
    """The multicore CPU baseline in the manner of Algorithm 2 (M-BBC:
    OpenMP over the smaller side's anchors, heaviest first, thread-local
    buckets, priority pair filter) on the whole graph with every host core;
    its total must equal the GPU's."""
    import oracle

    t0 = time.perf_counter()
    t, threads = oracle.mbbc_count(g)
    dt = time.perf_counter() - t0
    h = host_info()
    return dict(value=wedges / dt / 1e9, unit="G/s", seconds=dt, threads=threads, cores=h["cores"],
                model=h["model"], kind="multicore (Algorithm 2 style, OpenMP)", total_matches=bool(t == total),
                sample="whole graph, including its own CSR build and sorts")


def bench_copy(mib: int = 4096, reps: int = 5) -> dict:
    """Achievable HBM bandwidth on this device: a plain device-to-device
    copy of `mib` MiB (read + write bytes per second), timed by HIP events."""
    import torch

    n = mib << 20
    src = torch.ones(n, dtype=torch.uint8, device="cuda:0")
    dst = torch.empty_like(src)
    dst.copy_(src)
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(reps):
        dst.copy_(src)
    e1.record()
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / reps
    del src, dst
    torch.cuda.empty_cache()
    gbs = 2 * n / (ms / 1e3) / 1e9
    return dict(bytes_per_copy=2 * n, ms=ms, achieved=gbs, unit="GB/s", frac_of_peak=gbs / HBM_PEAK_GBS)


def bench_uniform(ctx, seed: int, calls: int = 200) -> dict:
    """Latency of one bbc_count call on the small uniform graph (|U| =
    2,000, |V| = 1,000, 20,000 edges, P(-) = 0.3): microseconds per call,
    host wait included, and the kernels' span by HIP events."""
    import torch

    from paper_2601_17707_amd import bbc, synth

    g = synth.workload("uniform-2k-1k-20k", seed)
    off, adj, sg = bbc.graph_tensors(g, "cuda:0")
    for _ in range(10):
        t = ctx.count(off, adj, sg, g.n_v)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(calls):
        t = ctx.count(off, adj, sg, g.n_v)
    us = 1e6 * (time.perf_counter() - t0) / calls
    span = []
    for _ in range(10):
        ctx.count(off, adj, sg, g.n_v, opts=bbc.options(timing=True))
        span.append(ctx.stats()["ms_total"])
    st = ctx.stats()
    return dict(workload="uniform-2k-1k-20k", seed=seed, n_edges=g.m, us_per_call=us,
                device_span_us=1e3 * sum(span) / len(span), kernel_us=1e3 * st["ms_count"], wedges=int(st["wedges"]),
                balanced_butterflies=t)


def bench_skewed(ctx, steps: int, warmup: int, seed: int, no_tune: bool = False) -> dict:
    """The highly skewed workload (|U| = 5e6, |V| = 2e5, 2e8 edges, hub V
    vertices near 430,000 edges): end-to-end, build and wedge-kernel times,
    wedges/s and the kernel's roofline fraction on algorithmic bytes, with
    the autotuner's configuration for this graph (tuning untimed) and the
    end-to-end time of the library's defaults beside it."""
    import torch

    from paper_2601_17707_amd import bbc, synth

    t0 = time.perf_counter()
    g = synth.workload("skewed-5m-200k-200m", seed)
    gen_s = time.perf_counter() - t0
    print(f"# skewed-5m-200k-200m: n_u={g.n_u} n_v={g.n_v} m={g.m} (generated in {gen_s:.1f} s)", file=sys.stderr,
          flush=True)
    off, adj, sg = bbc.graph_tensors(g, "cuda:0")
    n_v = g.n_v
    del g

    def time_calls(o):
        for _ in range(max(1, warmup)):
            tot = ctx.count(off, adj, sg, n_v, opts=o)
        torch.cuda.synchronize()
        t = time.perf_counter()
        for _ in range(steps):
            tot = ctx.count(off, adj, sg, n_v, opts=o)
        torch.cuda.synchronize()
        return tot, 1000.0 * (time.perf_counter() - t) / steps

    # defaults, then the autotuner on this graph (untimed), then its choice
    total_untuned, ms_untuned = time_calls(bbc.options(no_tuning=True))
    tuned = None if no_tune else ctx.autotune(off, adj, sg, n_v, reps=1)
    total, ms = time_calls(bbc.options())
    assert total == total_untuned
    kern, build = [], []
    for _ in range(3):
        ctx.count(off, adj, sg, n_v, opts=bbc.options(timing=True))
        st = ctx.stats()
        kern.append(st["ms_count"])
        build.append(st["ms_checks"] + st["ms_build"])
    kavg = sum(kern) / len(kern)
    wedges = int(st["wedges"])
    nbytes = algorithmic_bytes(st)
    ach = nbytes / (kavg / 1e3) / 1e9
    del off, adj, sg
    torch.cuda.empty_cache()
    return dict(workload="skewed-5m-200k-200m", seed=seed, n_edges=int(st["n_edges"]), wedges=wedges,
                ms_per_call=ms, ms_per_call_untuned=ms_untuned, tuned=tuned, kernel_ms=kavg,
                build_ms=sum(build) / len(build),
                wedges_per_s=wedges / (ms / 1e3) / 1e9, kernel_wedges_per_s=wedges / (kavg / 1e3) / 1e9, unit="G/s",
                balanced_butterflies=total, bands=int(st["bands"]),
                roofline=dict(bound="hbm", kernel="k_wedge", achieved=ach, peak=HBM_PEAK_GBS, unit="GB/s",
                              frac=ach / HBM_PEAK_GBS, algorithmic_bytes=nbytes))


def bench_batched(ctx, steps: int, warmup: int, seed: int) -> dict:
    """Graphs/s of the 10,000-graph batch: one captured batch plan replayed
    (inputs resident in HBM), tuned once for this batch by the autotuner
    (untimed; the untuned plan is timed too), against a loop of plain
    per-graph bbc_count calls on views of the same device arrays.  All must
    give identical per-graph totals."""
    import torch

    from paper_2601_17707_amd import bbc, synth

    t0 = time.perf_counter()
    graphs = synth.workload("batch-10k", seed)
    gen_s = time.perf_counter() - t0
    batch = bbc.Batch(graphs, "cuda:0")
    n = len(graphs)
    edges = sum(g.m for g in graphs)
    print(f"# batch-10k: {n} graphs, {edges} edges (generated in {gen_s:.1f} s)", file=sys.stderr, flush=True)
    def time_plan(opts):
        plan = ctx.plan(batch, opts=opts)
        for _ in range(max(1, warmup)):
            plan.launch()
            plan.wait()
        torch.cuda.synchronize()
        ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        t0 = time.perf_counter()
        ev0.record()
        for _ in range(steps):
            plan.launch()
        ev1.record()
        tot = plan.wait().cpu().numpy()[:n].copy()
        torch.cuda.synchronize()
        ms = 1000.0 * (time.perf_counter() - t0) / steps
        plan.close()
        return tot, ms, ev0.elapsed_time(ev1) / steps

    # untuned plan, then the autotuner on this batch (untimed), then the
    # tuned plan, which is the batch figure
    totals_untuned, ms_untuned, _ = time_plan(bbc.options(no_tuning=True))
    t0 = time.perf_counter()
    tuned = ctx.autotune_batched(batch, reps=1)
    tune_s = time.perf_counter() - t0
    totals, ms_batch, ms_batch_ev = time_plan(bbc.options())

    # aggregate rate of the batch: every graph's wedges, and the wedge
    # kernel's algorithmic bytes over its HIP-event time (one eager pass)
    ctx.count_batched(batch, opts=bbc.options(timing=True))
    bst = ctx.stats()
    b_wedges = int(bst["wedges"])
    b_bytes = algorithmic_bytes(bst)
    b_kern = bst["ms_count"]

    # per-graph loop: plain bbc_count on each graph's slice of the same arrays
    loop = [0] * n
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for i, d in enumerate(batch.descs[:n]):
        off = batch.offsets[d.off_base: d.off_base + d.n_u + 1]
        adj = batch.adj[d.edge_base: d.edge_base + d.n_edges]
        sg = batch.signs[d.edge_base: d.edge_base + d.n_edges]
        loop[i] = ctx.count(off, adj, sg, d.n_v)
    torch.cuda.synchronize()
    loop_s = time.perf_counter() - t0
    return dict(workload="batch-10k", graphs=n, edges=edges, ms_per_batch=ms_batch, ms_per_batch_events=ms_batch_ev,
                tuned=tuned, tune_s=tune_s, ms_per_batch_untuned=ms_untuned,
                totals_match_untuned=bool(list(totals) == list(totals_untuned)),
                graphs_per_s=n / (ms_batch / 1e3), per_graph_loop_s=loop_s, per_graph_loop_graphs_per_s=n / loop_s,
                speedup_vs_loop=(n / (ms_batch / 1e3)) / (n / loop_s),
                totals_match_loop=bool(list(totals) == loop), balanced_butterflies=int(totals.sum()),
                wedges=b_wedges, wedges_per_s=b_wedges / (ms_batch / 1e3) / 1e9, unit="G/s",
                kernel_ms=b_kern, build_ms=bst["ms_checks"] + bst["ms_build"],
                roofline=dict(bound="hbm", kernel="k_wedge", algorithmic_bytes=b_bytes,
                              achieved=b_bytes / (b_kern / 1e3) / 1e9, peak=HBM_PEAK_GBS, unit="GB/s",
                              frac=b_bytes / (b_kern / 1e3) / 1e9 / HBM_PEAK_GBS))


def bench_classes(ctx, off, adj, sg, n_v: int, wedges: int, total: int, steps: int, warmup: int) -> dict:
    """The six sign-pattern classes on the resident bench graph: the same
    wedges walked with three counters per endpoint.  The four balanced
    classes must add up to the balanced count."""
    import torch

    from paper_2601_17707_amd import bbc

    opts, opts_t = bbc.options(), bbc.options(timing=True)
    for _ in range(max(1, warmup)):
        ctx.count_classes(off, adj, sg, n_v, opts=opts)
    torch.cuda.synchronize()
    t = time.perf_counter()
    for _ in range(steps):
        cls = ctx.count_classes(off, adj, sg, n_v, opts=opts)
    torch.cuda.synchronize()
    ms = 1000.0 * (time.perf_counter() - t) / steps
    kern = []
    for _ in range(3):
        ctx.count_classes(off, adj, sg, n_v, opts=opts_t)
        kern.append(ctx.stats()["ms_count"])
    return dict(ms_per_call=ms, kernel_ms=sum(kern) / len(kern), wedges_per_s=wedges / (ms / 1e3) / 1e9, unit="G/s",
                classes=dict(zip(("pp_pp", "pp_mm", "mm_mm", "pm_pm", "pp_pm", "pm_mm"), cls)),
                balanced_matches_count=bool(sum(cls[:4]) == total))


def bench_bicliques(ctx, off, adj, sg, n_v: int, wedges: int, total: int, steps: int, warmup: int) -> dict:
    """Balanced (2,k)-bicliques on the resident bench graph with the pair on
    U, the size-two side the BB2K section fixes, for k = 3 and 4 (exact
    128-bit sums), and k = 2 checked against the balanced count.  Wedges
    are those of the U-anchored walk (sum of C(deg v, 2) over V)."""
    import torch

    from paper_2601_17707_amd import bbc

    out = {}
    for k in (2, 3, 4):
        for _ in range(max(1, warmup)):
            r = ctx.count_bicliques(off, adj, sg, n_v, k)
        torch.cuda.synchronize()
        t = time.perf_counter()
        for _ in range(steps):
            r = ctx.count_bicliques(off, adj, sg, n_v, k)
        torch.cuda.synchronize()
        ms = 1000.0 * (time.perf_counter() - t) / steps
        ctx.count_bicliques(off, adj, sg, n_v, k, opts=bbc.options(timing=True))
        bst = ctx.stats()
        w_k = int(bst["wedges"])
        out[f"k{k}"] = dict(count=str(r), ms_per_call=ms, kernel_ms=bst["ms_count"], wedges=w_k,
                            wedges_per_s=w_k / (ms / 1e3) / 1e9)
    out["unit"] = "G/s"
    out["pair_side"] = "U"
    out["k2_matches_count"] = bool(int(out["k2"]["count"]) == total)
    return out


def bench_updates(ctx, g, off, adj, sg, count_ms: float, steps: int, warmup: int, seed: int,
                  q: int = 100_000) -> dict:
    """A batch of q edge updates on the resident bench graph (half re-sign
    or remove existing edges, half add or leave absent pairs; states drawn
    from {-1, 0, +1}): the change of the count by bbc_update_delta, against
    the time of one full count.  The per-update shares must sum to it."""
    import numpy as np
    import torch

    dev = off.device
    rng = np.random.default_rng(seed + 100)
    pick = rng.choice(g.m, q // 2, replace=False)
    eu = np.searchsorted(g.offsets.astype(np.int64), pick, side="right") - 1
    keys = set((eu.astype(np.int64) * g.n_v + g.adj[pick]).tolist())
    while len(keys) < q:
        keys.add(int(rng.integers(0, g.n_u)) * g.n_v + int(rng.integers(0, g.n_v)))
    k = np.array(sorted(keys), np.int64)
    rng.shuffle(k)
    tu = torch.as_tensor((k // g.n_v).astype(np.int32), device=dev)
    tv = torch.as_tensor((k % g.n_v).astype(np.int32), device=dev)
    ts = torch.as_tensor(rng.choice([-1, 0, 1], size=q).astype(np.int8), device=dev)
    shares = torch.empty(q, dtype=torch.int64, device=dev)
    for _ in range(max(1, warmup)):
        d = ctx.update_delta(off, adj, sg, g.n_v, tu, tv, ts)
    torch.cuda.synchronize()
    t = time.perf_counter()
    for _ in range(steps):
        d = ctx.update_delta(off, adj, sg, g.n_v, tu, tv, ts)
    torch.cuda.synchronize()
    ms = 1000.0 * (time.perf_counter() - t) / steps
    d2 = ctx.update_delta(off, adj, sg, g.n_v, tu, tv, ts, per_update=shares)
    return dict(updates=q, ms_per_batch=ms, updates_per_s=q / (ms / 1e3), delta=d,
                shares_sum_match=bool(int(shares.sum()) == d == d2), full_count_ms=count_ms,
                speedup_vs_recount=count_ms / ms)


def bench_hybrid(ctx, steps: int, warmup: int, seed: int) -> dict:
    """The planted-block workload (power-law background, |U| = 2e6, |V| = 1e6,
    5e7 background edges, 16 blocks of 4096 x 4096 at density 0.5) counted
    with its blocks on int8 matrix cores, against the sparse-only path on the
    same resident graph.  Both totals must agree.  Effective wedges/s counts
    every wedge (dense ones included); the dense kernel's rate is int8
    operations (2 products x 2 ops per multiply-add, upper triangle) per
    second of its HIP-event duration."""
    import torch

    from paper_2601_17707_amd import bbc, synth

    dev = torch.device("cuda:0")
    t0 = time.perf_counter()
    g = synth.workload(HYBRID_WORKLOAD, seed)
    gen_s = time.perf_counter() - t0
    print(f"# {HYBRID_WORKLOAD}: n_u={g.n_u} n_v={g.n_v} m={g.m} (generated in {gen_s:.1f} s)", file=sys.stderr,
          flush=True)
    off, adj, sg = bbc.graph_tensors(g, dev)
    blocks = [(torch.from_numpy(c).to(dev), torch.from_numpy(r).to(dev)) for r, c in g.meta["blocks"]]
    opts_h, opts_ht = bbc.options(blocks=blocks), bbc.options(blocks=blocks, timing=True)
    opts_s = bbc.options()

    def timed_calls(opts, n):
        torch.cuda.synchronize()
        t = time.perf_counter()
        for _ in range(n):
            tot = ctx.count(off, adj, sg, g.n_v, opts=opts)
        torch.cuda.synchronize()
        return tot, 1000.0 * (time.perf_counter() - t) / n

    for _ in range(max(1, warmup)):
        ctx.count(off, adj, sg, g.n_v, opts=opts_h)
    total_h, ms_h = timed_calls(opts_h, steps)
    dense_ms, count_ms = [], []
    for _ in range(3):
        ctx.count(off, adj, sg, g.n_v, opts=opts_ht)
        st = ctx.stats()
        dense_ms.append(st["ms_dense"])
        count_ms.append(st["ms_count"])
    ops = int(st["dense_ops"])
    dms = sum(dense_ms) / len(dense_ms)
    ctx.count(off, adj, sg, g.n_v, opts=opts_s)
    total_s, ms_s = timed_calls(opts_s, max(1, min(steps, 3)))
    # the same graph with blocks found by the planner instead of the planted list
    torch.cuda.synchronize()
    t = time.perf_counter()
    found = ctx.plan_blocks(off, adj, g.n_v)
    plan_ms = 1000.0 * (time.perf_counter() - t)
    opts_p = bbc.options(blocks=found)
    ctx.count(off, adj, sg, g.n_v, opts=opts_p)
    total_p, ms_p = timed_calls(opts_p, max(1, min(steps, 3)))
    tops = ops / (dms / 1e3) / 1e12
    return dict(workload=HYBRID_WORKLOAD, seed=seed, n_u=g.n_u, n_v=g.n_v, n_edges=g.m, blocks="16 x (4096 x 4096)",
                wedges=int(st["wedges_all"]), wedges_sparse_walk=int(st["wedges"]),
                ms_per_call=ms_h, ms_per_call_sparse_only=ms_s, speedup_vs_sparse_only=ms_s / ms_h,
                effective_wedges_per_s=int(st["wedges_all"]) / (ms_h / 1e3) / 1e9, unit="G/s",
                count_ms=sum(count_ms) / len(count_ms),
                dense=dict(kernel="k_dense", ms=dms, int8_ops=ops, achieved=tops, peak=INT8_PEAK_TOPS, unit="TOP/s",
                           frac=tops / INT8_PEAK_TOPS, bound="mfma"),
                balanced_butterflies=total_h, totals_match_sparse_only=bool(total_h == total_s),
                planner=dict(ms=plan_ms, blocks=len(found), ms_per_call=ms_p, speedup_vs_sparse_only=ms_s / ms_p,
                             totals_match=bool(total_p == total_s)))


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--workload", default=WORKLOAD)
    ap.add_argument("--seed", type=int, default=1)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-batch", action="store_true", help="skip the 10,000-graph batch measurement")
    ap.add_argument("--no-tune", action="store_true",
                    help="time the library's default configuration (no autotuning of the main graph)")
    ap.add_argument("--save-tune", default="", help="write the tuning table after autotuning the main graph")
    ap.add_argument("--tune-file", default="",
                    help="load this tuning table instead of autotuning (profiled runs: the tuned configuration "
                         "without the tuning launches; the default-configuration steps still run unless --no-tune)")
    ap.add_argument("--no-hybrid", action="store_true", help="skip the dense-block workload")
    ap.add_argument("--no-classes", action="store_true", help="skip the sign-pattern class count")
    ap.add_argument("--no-bicliques", action="store_true", help="skip the (2,k)-biclique counts")
    ap.add_argument("--no-updates", action="store_true", help="skip the dynamic-update batch")
    ap.add_argument("--no-skewed", action="store_true", help="skip the 200M-edge skewed workload")
    ap.add_argument("--no-uniform", action="store_true", help="skip the small-graph latency measurement")
    ap.add_argument("--no-multicore", action="store_true", help="skip the multicore CPU baseline")
    ap.add_argument("--no-copy", action="store_true", help="skip the device copy bandwidth measurement")
    ap.add_argument("--copy-probe-mib", type=int, default=0,
                    help="first run one plain device-to-device copy of this many MiB (a known-size "
                         "reference for hardware byte counters)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(json.dumps(dict(error="this benchmark runs on one GPU only; multi-GPU sharding is not built",
                              n_gpus=args.gpus)), flush=True)
        sys.exit(2)

    import torch

    import __graft_entry__

    __graft_entry__._ensure_built()
    from paper_2601_17707_amd import bbc, synth

    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    t0 = time.perf_counter()
    g = synth.workload(args.workload, args.seed)
    gen_s = time.perf_counter() - t0
    print(f"# workload {args.workload} seed {args.seed}: n_u={g.n_u} n_v={g.n_v} m={g.m} "
          f"(generated in {gen_s:.1f} s)", file=sys.stderr, flush=True)
    ctx = bbc.Context(0)
    off, adj, sg = bbc.graph_tensors(g, dev)
    if args.copy_probe_mib > 0:
        n = args.copy_probe_mib << 20
        src = torch.ones(n, dtype=torch.uint8, device=dev)
        dst = torch.empty_like(src)
        torch.cuda.synchronize()
        dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst
    opts_t = bbc.options(timing=True)
    opts = bbc.options()

    def time_steps(o):
        for _ in range(args.warmup):
            t = ctx.count(off, adj, sg, g.n_v, opts=o)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(args.steps):
            t = ctx.count(off, adj, sg, g.n_v, opts=o)
        torch.cuda.synchronize()
        return t, 1000.0 * (time.perf_counter() - t0) / args.steps

    # the library's defaults first, then the autotuner on this graph
    # (untimed; it records the fastest configuration for the graph's size
    # class, which later calls with default options use), then the timed
    # steps with that configuration
    total_untuned, ms_untuned = (None, None) if args.no_tune else time_steps(bbc.options(no_tuning=True))
    tuned, tune_s = None, None
    if args.tune_file:  # a table an earlier run saved: same configuration, no tuning launches
        ctx.tune_load(args.tune_file)
    elif not args.no_tune:
        t0 = time.perf_counter()
        tuned = ctx.autotune(off, adj, sg, g.n_v, reps=1)
        tune_s = time.perf_counter() - t0
        print(f"# autotuned in {tune_s:.1f} s: {tuned}", file=sys.stderr, flush=True)
        if args.save_tune:
            ctx.tune_save(args.save_tune)
    total, ms_step = time_steps(opts)
    assert total_untuned is None or total_untuned == total

    # kernel durations from HIP events recorded on the launch stream
    kern_ms, build_ms = [], []
    for _ in range(max(3, min(args.steps, 10))):
        t = ctx.count(off, adj, sg, g.n_v, opts=opts_t)
        assert t == total
        st = ctx.stats()
        kern_ms.append(st["ms_count"])
        build_ms.append(st["ms_checks"] + st["ms_build"])
    st = ctx.stats()
    wedges = int(st["wedges"])
    kavg = sum(kern_ms) / len(kern_ms)
    two_sided = max(g.n_u, g.n_v) <= 8 * min(g.n_u, g.n_v) and g.m ** 2 <= 64 ** 2 * g.n_u * g.n_v
    walked = two_sided_wedges(g) if two_sided else wedges
    nbytes = two_sided_bytes(g, walked) if two_sided else algorithmic_bytes(st)
    achieved = nbytes / (kavg / 1e3) / 1e9

    line = dict(
        metric="wedges/sec",
        value=wedges / (ms_step / 1e3) / 1e9,
        unit="G/s",
        n_gpus=1,
        steps=args.steps,
        warmup=args.warmup,
        ms_per_step=ms_step,
        higher_is_better=True,
        scaling="weak",
        vs_baseline=None,
        dtype="u32",
        data="synthetic",
        config=dict(workload=args.workload, seed=args.seed, n_u=g.n_u, n_v=g.n_v, n_edges=g.m,
                    anchor_side="U" if st["side"] == bbc.SIDE_U else "V", wedges=wedges),
        balanced_butterflies=total,
        balanced_butterflies_per_s=total / (ms_step / 1e3),
        kernel_ms=kavg,
        build_ms=sum(build_ms) / len(build_ms),
        kernel_wedges_per_s=wedges / (kavg / 1e3) / 1e9,
        wedges_walked=walked,
        kernel_wedges_walked_per_s=walked / (kavg / 1e3) / 1e9,
        tuned=tuned,
        tune_s=tune_s,
        ms_per_step_untuned=ms_untuned,
        value_untuned=None if ms_untuned is None else wedges / (ms_untuned / 1e3) / 1e9,
        roofline=dict(bound="hbm", achieved=achieved, peak=HBM_PEAK_GBS, unit="GB/s", frac=achieved / HBM_PEAK_GBS,
                      traffic=measured_traffic(args.workload),
                      kernel="k_top_bands + k_top_hash + k_top_light" if two_sided else "k_wedge",
                      algorithmic_bytes=nbytes,
                      bands=int(st["bands"])),
    )
    if not args.no_classes:
        line["classes"] = bench_classes(ctx, off, adj, sg, g.n_v, wedges, total, max(1, min(args.steps, 5)),
                                        args.warmup)
    if not args.no_bicliques:
        line["bicliques"] = bench_bicliques(ctx, off, adj, sg, g.n_v, wedges, total, max(1, min(args.steps, 3)),
                                            args.warmup)
    if not args.no_updates:
        line["updates"] = [bench_updates(ctx, g, off, adj, sg, ms_step, max(1, min(args.steps, 5)), args.warmup,
                                         args.seed, q=q) for q in (1_000, 100_000)]
    if not args.no_uniform and args.workload == WORKLOAD:
        line["uniform"] = bench_uniform(ctx, args.seed)
    if not args.no_batch and args.workload == WORKLOAD:
        line["batched"] = bench_batched(ctx, max(1, min(args.steps, 5)), args.warmup, args.seed)
    if args.workload == WORKLOAD and not (args.no_hybrid and args.no_skewed):
        del off, adj, sg
        torch.cuda.empty_cache()
    if not args.no_hybrid and args.workload == WORKLOAD:
        line["hybrid"] = bench_hybrid(ctx, max(1, min(args.steps, 5)), args.warmup, args.seed)
    if not args.no_skewed and args.workload == WORKLOAD:
        line["skewed"] = bench_skewed(ctx, max(1, min(args.steps, 3)), args.warmup, args.seed, args.no_tune)
    if not args.no_copy:
        line["hbm_copy"] = bench_copy()
    line["host"] = host_info()
    if not args.no_cpu_baseline:
        line["cpu_baseline"] = cpu_baseline(g, wedges)
    if not args.no_multicore:
        line["cpu_multicore"] = cpu_multicore(g, wedges, total)
    ctx.close()
    print(json.dumps(line), flush=True)


if __name__ == "__main__":
    main()
