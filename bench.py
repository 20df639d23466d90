#!/usr/bin/env python3
"""Throughput benchmark of the sampling triangle counter on one MI355X.

Workload (default): R-MAT scale 22, edge factor 16 (a/b/c = .57/.19/.19, no
noise, seeded relabelling, generator seed 1), symmetrised and cleaned into an
int32 CSR that stays resident in HBM.  One step is the whole counting path at
the four operating points of that workload: the exact count (p = 1) and the
sparsify-then-count estimates at p = 0.5, 0.1 and 0.05 with seed 0 (each:
hash coin, degree orientation, light/heavy split, light wedge closure, heavy
int8-MFMA block, rescale).  The metric is sampled-graph edges per second: the
edges of the four counted graphs (m, m'_0.5, m'_0.1, m'_0.05) divided by the
step time.  The CSR build is timed separately (the paper also leaves the
conversion to its sorted-list format out of its timings, section 4.2).
Before timing, the autotuner picks per operating point the launch parameters
and the heavy multiplier c (light iff deg <= c sqrt(m'), c in {1/4, 1/2, 1,
2}) on a different sample (seed + 1); the count is the same for every c.
--defaults times the paper's split (c = 1) with default launch parameters.

Prints one JSON line.  Only one GPU is supported.
"""
import argparse
import hashlib
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0
# serving: requests of at most this many pairs (R-MAT scale <= 14 at edge
# factor 16) are fused with the small requests queued behind them
FUSE_PAIRS = 1 << 18
# the list kernels of the light closure, by the model their items are counted in
LIGHT_KERNELS = {"light_small": ("light_small",), "light_large": ("light_bits", "light_large", "light_huge")}


def _light_model_bytes(c, large):
    """Bytes a light-closure kernel must read under the list model, as counted
    by the library: per work item the anchor's row offsets and its staged
    out-list (4 B per entry); per iterated entry the entry and the row offsets
    of its list; per probe the streamed list entry (4 B).  The bitmap kernel
    reads names of 2 B in their place, so for it the model is no byte rate."""
    return c["model_bytes_large"] if large else c["model_bytes_small"]


COUNT_SOURCES = ("tc_count.hip", "tc_device.h")
STREAM_SOURCES = ("tc_stream.hip", "tc_prefix.h", "tc_device.h")


def _source_sha(sources=COUNT_SOURCES):
    """Hash of the sources a kernel is compiled from (default: the counting kernels)."""
    h = hashlib.sha256()
    for name in sources:
        with open(os.path.join(ROOT, "paper_1011_0468_amd", "csrc", name), "rb") as f:
            h.update(f.read())
    return h.hexdigest()[:16]


def _traffic(kernel, workload, tunings, sources=COUNT_SOURCES):
    """HBM bytes per launch from committed rocprofv3 counter runs, if they were
    taken on the current kernel source with the same launch parameters."""
    path = os.path.join(ROOT, "profiles", "%s_%s_traffic.json" % (kernel, workload))
    if not os.path.exists(path):
        return None
    try:
        rec = json.load(open(path))
    except Exception:
        return None
    if rec.get("source_sha") != _source_sha(sources) or rec.get("tunings") != tunings:
        return None
    return rec.get("hbm_bytes_per_launch")


def _cpu_model():
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def cpu_baseline(workload, ps, seeds, gpu_ms=None):
    """The oracle (single-threaded C, this thread pinned to one core) on a
    bounded sample of the same workload: sampling plus exact split count of
    each sampled graph, for the operating points ps and the sample seeds.
    gpu_ms (p -> ms of one call) gives the device's rate on the same legs."""
    import oracle
    import synth
    g = oracle.normalise(*synth.workload(workload))
    allowed = sorted(os.sched_getaffinity(0))
    pin = allowed[0]
    os.sched_setaffinity(0, {pin})
    try:
        edges, secs, counts = 0, 0.0, {}
        for p in ps:
            for sd in seeds:
                t = time.perf_counter()
                gp = oracle.sample(g, p, sd)
                r = oracle.count_split(gp, 1, 1)
                secs += time.perf_counter() - t
                edges += r["m"]
                counts[(p, sd)] = r
    finally:
        os.sched_setaffinity(0, set(allowed))
    out = {"value": edges / secs, "unit": "edges/s", "cores": 1, "kind": "oracle",
           "sample": "%s, p in %s, seeds %s: oracle sample + exact split count of each sampled graph "
                     "(%.1f s on one pinned core; the p=1 and p=0.5 legs take minutes and are left out)"
                     % (workload, list(ps), list(seeds), secs),
           "pinned_cpu": pin, "nproc": len(allowed), "cpu_model": _cpu_model()}
    if gpu_ms:
        # the device on the same legs (seed 0 calls, per-call wall time)
        e0 = sum(counts[(p, seeds[0])]["m"] for p in ps)
        t0 = sum(gpu_ms[p] for p in ps) / 1e3
        out["gpu_same_legs_edges_per_s"] = e0 / t0
    return out, counts


def batched(args):
    """Batched trials: Chung-Lu n=2^20 (avg degree 32, beta 2.2), seeds 0..63 at
    p = 0.05 in one batched call with median of 8 means, against 64 single-seed
    calls on the same graph.  Throughput = sum of sampled edges / time."""
    import torch
    import synth
    import paper_1011_0468_amd as tc
    n, s, d = synth.workload("cl20")
    g = tc.tc_build_csr(n, torch.from_numpy(s).cuda(), torch.from_numpy(d).cuda())
    seeds = list(range(64))
    p = 0.05

    def one_batch():
        return tc.tc_estimate(g, p, seeds, num_groups=8)

    def singles():
        return [tc.tc_estimate(g, p, [sd])[0][0] for sd in seeds]

    for _ in range(args.warmup):
        one_batch()
        singles()
    torch.cuda.synchronize()
    t = time.perf_counter()
    for _ in range(args.steps):
        per, ests, mom = one_batch()
    torch.cuda.synchronize()
    ms_batch = (time.perf_counter() - t) * 1e3 / args.steps
    t = time.perf_counter()
    for _ in range(args.steps):
        one = singles()
    torch.cuda.synchronize()
    ms_single = (time.perf_counter() - t) * 1e3 / args.steps
    edges = sum(c["m"] for c in per)
    assert [c["triangles"] for c in per] == [c["triangles"] for c in one]

    # the heavy multipliers c in {1/2, 1, 2} and the autotuner's choice (tuned
    # on seed 1000, which is not in the batch), each timed on the same batch:
    # the counts must not change, only the reported light/heavy split
    def timed_batch(**kw):
        for _ in range(max(1, args.warmup)):
            tc.tc_estimate(g, p, seeds, num_groups=8, **kw)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(args.steps):
            pv, _, mv = tc.tc_estimate(g, p, seeds, num_groups=8, **kw)
        torch.cuda.synchronize()
        assert [c["triangles"] for c in pv] == [c["triangles"] for c in per] and mv == mom
        return round((time.perf_counter() - t0) * 1e3 / args.steps, 3), sum(c["n_heavy"] for c in pv)
    variants = {}
    for a, b in ((1, 2), (1, 1), (2, 1)):
        ms_v, nh = timed_batch(heavy=(a, b))
        variants["%d/%d" % (a, b)] = {"ms": ms_v, "heavy_vertices_all_seeds": nh}
    choice = tc.tc_autotune(g, p, seed=1000)
    ms_t, nh_t = timed_batch(tuned=True)
    variants["autotuned"] = {"ms": ms_t, "heavy_vertices_all_seeds": nh_t, "choice": choice}
    print(json.dumps({"metric": "batched sampled-graph edges/sec (64 seeds, one call)", "value": edges / (ms_batch / 1e3),
                      "unit": "edges/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
                      "ms_per_step": round(ms_batch, 3), "ms_64_single_calls": round(ms_single, 3),
                      "speedup_vs_single_calls": round(ms_single / ms_batch, 2), "median_of_means": mom,
                      "heavy_multiplier_runs": variants,
                      "higher_is_better": True, "dtype": "int32", "data": "synthetic",
                      "config": {"workload": "cl20", "n": n, "m": g.info()["m"], "p": p, "seeds": 64, "groups": 8}}),
          flush=True)


def latency_cl16k(args):
    """Latency of the small configuration, Chung-Lu n = 16384 (avg degree 12,
    beta 2.5): the exact count and the p = 0.25 estimate of seed 0, each call
    timed on its own (it synchronises its stream) over 50 calls after 5
    warm-up calls: median, min and max in microseconds.  Counts against the
    oracle's stored values; the oracle's own time on the same two calls."""
    import statistics
    import torch
    import synth
    import paper_1011_0468_amd as tc
    n, s, d = synth.workload("cl16k")
    g = tc.tc_build_csr(n, torch.from_numpy(s).cuda(), torch.from_numpy(d).cuda())
    reps = max(50, args.steps)
    calls = {"exact": lambda: tc.tc_count_exact(g),
             "p=0.25": lambda: tc.tc_estimate(g, 0.25, [0])[0][0]}
    out, got = {}, {}
    for name, fn in calls.items():
        for _ in range(max(5, args.warmup)):
            fn()
        torch.cuda.synchronize()
        us = []
        for _ in range(reps):
            t0 = time.perf_counter()
            got[name] = fn()
            us.append((time.perf_counter() - t0) * 1e6)
        out[name] = {"median_us": round(statistics.median(us), 1), "min_us": round(min(us), 1),
                     "max_us": round(max(us), 1), "calls": reps}
    golden = _load_golden("cl16k.json")
    parity = None
    if golden:
        want = {c["p"]: c for c in golden["counts"]}
        keys = ("triangles", "light", "heavy", "n_heavy", "m")
        parity = all(got[name][k] == want[p][k] for name, p in (("exact", 1.0), ("p=0.25", 0.25)) for k in keys)
    line = {"metric": "latency of the exact count on Chung-Lu n=16384 (one call, median)",
            "value": out["exact"]["median_us"], "unit": "us", "n_gpus": 1, "steps": reps, "warmup": max(5, args.warmup),
            "higher_is_better": False, "dtype": "int32", "data": "synthetic", "calls": out,
            "parity_vs_oracle": parity, "config": {"workload": "cl16k", "n": n, "m": g.info()["m"]}}
    if not args.no_cpu_baseline:
        line["cpu_baseline"] = cpu_baseline_calls("cl16k", ((1.0, 0), (0.25, 0)), reps=20)
    print(json.dumps(line), flush=True)


def cpu_baseline_calls(workload, legs, reps):
    """The oracle (one pinned core) on the given (p, seed) legs, repeated reps
    times: median microseconds per leg (sampling plus exact split count)."""
    import statistics
    import oracle
    import synth
    g = oracle.normalise(*synth.workload(workload))
    allowed = sorted(os.sched_getaffinity(0))
    pin = allowed[0]
    os.sched_setaffinity(0, {pin})
    try:
        res = {}
        for p, sd in legs:
            us = []
            for _ in range(reps):
                t0 = time.perf_counter()
                gp = g if p == 1.0 else oracle.sample(g, p, sd)
                oracle.count_split(gp, 1, 1)
                us.append((time.perf_counter() - t0) * 1e6)
            res["p=%g" % p] = round(statistics.median(us), 1)
    finally:
        os.sched_setaffinity(0, set(allowed))
    return {"value": res["p=1"], "unit": "us", "cores": 1, "kind": "oracle", "per_leg_median_us": res,
            "sample": "%s: the exact count and the p=0.25 sample + count of seed 0, %d times each, median"
                      % (workload, reps), "pinned_cpu": pin, "nproc": len(allowed), "cpu_model": _cpu_model()}


def adaptive(args):
    """Adaptive keep probability on R-MAT scale 22: p doubles from 1/64 with 16
    seeds per stage (median of 4 means) until two stages agree to 1%; the time
    of the whole search, its stages, the balance point of section 3.3 and the
    error against the exact count (measured once, outside the timed region)."""
    import torch
    import synth
    import paper_1011_0468_amd as tc
    n, s, d = synth.workload("rmat22")
    g = tc.tc_build_csr(n, torch.from_numpy(s).cuda(), torch.from_numpy(d).cuda())
    T = tc.tc_count_exact(g)["triangles"]
    p0, tol, S, G = 1 / 64, 0.01, 16, 4

    def search():
        return tc.tc_estimate_adaptive(g, p0, tol, args.seed, S, G)

    for _ in range(args.warmup):
        search()
    torch.cuda.synchronize()
    t = time.perf_counter()
    for _ in range(args.steps):
        stages, pb = search()
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t) * 1e3 / args.steps
    edges = sum(x["m_sum"] for x in stages)
    print(json.dumps({"metric": "adaptive-p search time (1 MI355X) at R-MAT s22", "value": round(ms, 3), "unit": "ms",
                      "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "higher_is_better": False,
                      "dtype": "int32", "data": "synthetic", "edges_per_s": edges / (ms / 1e3),
                      "p_chosen": stages[-1]["p"], "estimate": stages[-1]["estimate"], "exact": T,
                      "rel_error": stages[-1]["estimate"] / T - 1.0, "p_balance": pb,
                      "stages": [[x["p"], x["estimate"], x["m_sum"]] for x in stages],
                      "config": {"workload": "rmat22", "n": n, "m": g.info()["m"], "p0": p0, "tol": tol,
                                 "seeds_per_stage": S, "groups": G, "seed0": args.seed}}), flush=True)


def triples(args):
    """Triple sampling on R-MAT scale 22, the layout of Table 2: Simple and
    Hybrid, unsparsified and sparsified (p = 0.1), with m' samples (as many
    closure queries as edges); time per call and error against the exact
    count (measured once, outside the timed region)."""
    import torch
    import synth
    import paper_1011_0468_amd as tc
    n, s, d = synth.workload("rmat22")
    g = tc.tc_build_csr(n, torch.from_numpy(s).cuda(), torch.from_numpy(d).cuda())
    T = tc.tc_count_exact(g)["triangles"]
    m = g.info()["m"]
    rows = []
    for p in (1.0, 0.1):
        S = int(m * p)
        for hybrid in (False, True):
            def call():
                return tc.tc_triple_estimate(g, p, S, hybrid=hybrid, sample_seed=args.seed, triple_seed=args.seed + 1)
            for _ in range(args.warmup):
                call()
            torch.cuda.synchronize()
            t = time.perf_counter()
            for _ in range(args.steps):
                r = call()
            torch.cuda.synchronize()
            ms = (time.perf_counter() - t) * 1e3 / args.steps
            rows.append({"variant": "hybrid" if hybrid else "simple", "p": p, "samples": S, "ms": round(ms, 3),
                         "U": r["size"], "closed": r["closed"], "estimate": r["estimate"],
                         "err_pct": round(100.0 * abs(r["estimate"] / T - 1.0), 4),
                         "samples_per_s": S / (ms / 1e3)})
    print(json.dumps({"metric": "triple-sampling estimates (1 MI355X) at R-MAT s22", "value": rows[0]["ms"], "unit": "ms",
                      "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "higher_is_better": False,
                      "dtype": "int32", "data": "synthetic", "exact": T, "rows": rows,
                      "config": {"workload": "rmat22", "n": n, "m": m, "samples": "m' per call",
                                 "seed": args.seed}}), flush=True)


def serving_trace(N, loads=(0.5, 0.8, 0.95), pinned=True, log=True):
    """Serving: N R-MAT requests (scale uniform in [10, 20], edge factor 16,
    generator seed 1000 + i) counted at p uniform in {1, .5, .1} (sample seed
    i) by the serving engine with an 8 GiB arena.  The one-at-a-time capacity
    is measured closed-loop; then Poisson arrivals (seed 12345) at each load
    factor x that capacity are served by 4 lanes and by 1 lane (one request at
    a time, arrival order: one launch sequence per request) on the same trace.
    Latency = result ready - arrival; every request's counts must be identical
    in every run.  Returns the summary dict."""
    import concurrent.futures as cf
    import numpy as np
    import synth
    import paper_1011_0468_amd as tc

    scales, ps = synth.serving_requests(N)
    reqs = [None] * N
    t = time.perf_counter()
    with cf.ThreadPoolExecutor(max_workers=16) as ex:  # the generator releases the GIL
        futs = {ex.submit(synth.serving_graph, i, scales[i]): i for i in range(N)}
        for k, f in enumerate(cf.as_completed(futs)):
            reqs[futs[f]] = f.result()
            if log and (k + 1) % 200 == 0:
                print("generated %d/%d requests (%.1f s)" % (k + 1, N, time.perf_counter() - t),
                      file=sys.stderr, flush=True)
    pairs = int(sum(len(r[1]) for r in reqs))
    budget = 8 << 30
    keep = []
    if pinned:
        # request payloads in page-locked host memory, as a serving front end
        # would keep them: the copies to the device then run at DMA speed
        import torch
        for i, (n, s, d) in enumerate(reqs):
            ps_ = torch.empty(len(s), dtype=torch.int32, pin_memory=True)
            pd_ = torch.empty(len(d), dtype=torch.int32, pin_memory=True)
            ps_.numpy()[:] = s
            pd_.numpy()[:] = d
            keep.append((ps_, pd_))
            reqs[i] = (n, ps_.numpy(), pd_.numpy())

    def run(lanes, arrivals, fuse=0):
        with tc.Server(budget, lanes=lanes, fuse_max_pairs=fuse) as sv:
            t0 = sv.clock() + 0.05
            for i, (n, s, d) in enumerate(reqs):
                sv.submit(i, float(ps[i]), i, arrival_s=t0 + (arrivals[i] if arrivals is not None else 0.0),
                          n=n, src=s, dst=d)
            res = sv.drain()
            st = sv.stats()
        assert len(res) == N and all(x["status"] == 0 for x in res), [x["message"] for x in res if x["status"]][:3]
        assert st["spilled_bytes"] == 0
        res.sort(key=lambda x: x["id"])
        lat = np.array([x["done_s"] - x["arrival_s"] for x in res]) * 1e3
        span = max(x["done_s"] for x in res) - min(x["arrival_s"] for x in res)
        edges = sum(x["counts"]["m"] for x in res)
        out = {"lanes": lanes, "fuse_max_pairs": fuse, "p50_ms": round(float(np.percentile(lat, 50)), 3),
               "p99_ms": round(float(np.percentile(lat, 99)), 3), "req_per_s": round(N / span, 2),
               "edges_per_s": edges / span, "span_s": round(span, 3), "arena_peak": st["arena_peak"]}
        if log:
            print("lanes %d: %s" % (lanes, json.dumps(out)), file=sys.stderr, flush=True)
        return out, [x["counts"] for x in res]

    closed1, ref = run(1, None)
    closed4, c4 = run(4, None)
    assert c4 == ref
    closedf, cf_ = run(4, None, FUSE_PAIRS)
    assert cf_ == ref
    mu1 = closed1["req_per_s"]
    out_loads = {}
    for f in loads:
        arr = synth.poisson_arrivals(N, f * mu1, 12345)
        r4, c = run(4, arr)
        assert c == ref
        rf, c = run(4, arr, FUSE_PAIRS)
        assert c == ref
        r1, c = run(1, arr)
        assert c == ref
        out_loads[str(f)] = {"lambda_req_per_s": round(f * mu1, 2), "lanes4": r4, "fused": rf, "fifo": r1}
    return {"requests": N, "pairs": pairs,
            "capacity_req_per_s": {"fifo": mu1, "lanes4": closed4["req_per_s"], "fused": closedf["req_per_s"]},
            "closed_loop": {"fifo": closed1, "lanes4": closed4, "fused": closedf}, "loads": out_loads,
            "fuse_max_pairs": FUSE_PAIRS,
            "identical_alone_and_in_mix": True, "host_payloads": "pinned" if pinned else "pageable",
            "budget_bytes": budget, "arrival_seed": 12345}


def serve(args):
    """--workload serve: the full 1000-request trace at 0.5, 0.8, 0.95 x capacity."""
    import synth
    r = serving_trace(args.requests, pinned=not args.pageable)
    head = r["loads"]["0.8"]
    print(json.dumps({"metric": "serving p99 latency at 0.8 x one-at-a-time capacity", "value": head["fused"]["p99_ms"],
                      "unit": "ms", "n_gpus": 1, "higher_is_better": False, "dtype": "int32", "data": "synthetic",
                      "lanes4_p99_ms": head["lanes4"]["p99_ms"], "fifo_p99_ms": head["fifo"]["p99_ms"],
                      "fuse_max_pairs": r["fuse_max_pairs"], "capacity_req_per_s": r["capacity_req_per_s"],
                      "closed_loop": r["closed_loop"], "loads": r["loads"],
                      "identical_alone_and_in_mix": True, "host_payloads": r["host_payloads"],
                      "config": {"workload": "serve", "requests": r["requests"], "pairs": r["pairs"],
                                 "scales": [10, 20], "ps": list(synth.SERVE_P), "budget_bytes": r["budget_bytes"],
                                 "arrival_seed": 12345}}),
          flush=True)


def top_degree_subgraph(n, src, dst, deg, h):
    """Pairs of the subgraph induced by the h vertices of largest (degree, id),
    relabelled 0..h-1 in that order."""
    import numpy as np
    order = np.lexsort((np.arange(n), deg))[::-1][:h]
    lab = np.full(n, -1, np.int64)
    lab[order] = np.arange(h)
    keep = (lab[src] >= 0) & (lab[dst] >= 0)
    return lab[src[keep]].astype(np.int32), lab[dst[keep]].astype(np.int32)


def heavy_stress(args):
    """MFMA stress shape: the subgraph induced by the h highest-degree vertices
    of R-MAT s24 (h = 4096, 8192, 16384), counted with every vertex heavy
    (heavy_num = 0), so the whole count runs through the int8-MFMA block; the
    count is checked against the light/heavy split count of the same graph.
    Ops: the oriented form does one multiply-add per triple i < k < j,
    h^3/3 ops; the kernel executes 2 * 128^2 * 128 (J - I + 1) ops per macro
    tile I <= J."""
    import numpy as np
    import torch
    import synth
    import paper_1011_0468_amd as tc
    n, s, d = synth.workload("rmat24")
    g = tc.tc_build_csr(n, torch.from_numpy(s).cuda(), torch.from_numpy(d).cuda())
    _, _, deg = g.read()
    g.free()
    torch.cuda.empty_cache()
    rows = []
    for h in (4096, 8192, 16384):
        hs, hd = top_degree_subgraph(n, s, d, deg.astype(np.int64), h)
        sg = tc.tc_build_csr(h, torch.from_numpy(hs).cuda(), torch.from_numpy(hd).cuda())
        m = sg.info()["m"]
        ref = tc.tc_count_exact(sg)
        c = tc.tc_count_exact(sg, heavy=(0, 1))
        assert c["triangles"] == ref["triangles"] and c["light"] == 0
        tc.profile.select(["heavy_mfma"])
        tc.profile.reset()
        tc.profile.enable(True)
        for _ in range(args.steps):
            tc.tc_count_exact(sg, heavy=(0, 1))
        torch.cuda.synchronize()
        tc.profile.enable(False)
        ms_tot, launches = tc.profile.read("heavy_mfma")
        ms = ms_tot / launches
        hh = c["n_heavy"]
        nm = (hh + 127) // 128
        executed = 2 * 128 ** 3 * sum(J - I + 1 for J in range(nm) for I in range(J + 1))
        oriented = hh ** 3 / 3.0
        row = {"h": h, "n_heavy": hh, "m": m, "triangles": c["triangles"], "mfma_ms": round(ms, 4),
               "tops_oriented": round(oriented / (ms / 1e3) / 1e12, 1),
               "tops_executed": round(executed / (ms / 1e3) / 1e12, 1)}
        row["frac_executed"] = round(row["tops_executed"] / 5000.0, 4)
        print("heavy h=%d: %s" % (h, json.dumps(row)), file=sys.stderr, flush=True)
        rows.append(row)
        sg.free()
    top = rows[-1]
    print(json.dumps({"metric": "int8-MFMA heavy block throughput (top-16384 of R-MAT s24, all heavy)",
                      "value": top["tops_executed"], "unit": "TOP/s", "n_gpus": 1, "steps": args.steps,
                      "higher_is_better": True, "dtype": "i8", "data": "synthetic",
                      "roofline": {"bound": "mfma", "achieved": top["tops_executed"], "peak": 5000.0,
                                   "unit": "TFLOP/s", "frac": top["frac_executed"], "traffic": None,
                                   "kernel": "heavy_mfma"},
                      "shapes": rows, "config": {"workload": "heavy_stress", "graph": "rmat24", "h": [4096, 8192, 16384]}}),
          flush=True)


def rp_workload(args):
    """Random-projection trace on R-MAT scale 24 (k = 256 Rademacher vectors,
    seed 0): time per call, the sweeps' model bytes (CSR read twice per
    64-vector sweep plus the Y rows written and gathered) and the relative
    error of the estimate against the exact count (measured once, untimed)."""
    import torch
    import synth
    import paper_1011_0468_amd as tc
    n, s, d = synth.workload("rmat24")
    g = tc.tc_build_csr(n, torch.from_numpy(s).cuda(), torch.from_numpy(d).cuda())
    del s, d
    info = g.info()
    k = 256
    for _ in range(args.warmup):
        tc.tc_rp_trace(g, k, args.seed)
    tc.profile.select([])
    tc.profile.reset()
    tc.profile.enable(True)
    torch.cuda.synchronize()
    t = time.perf_counter()
    for _ in range(args.steps):
        q, est = tc.tc_rp_trace(g, k, args.seed)
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t) * 1e3 / args.steps
    tc.profile.enable(False)
    kern = {}
    for name in ("rp_spmm", "rp_dot", "rp_bound", "rp_clear"):
        tot, cnt = tc.profile.read(name)
        if cnt:
            kern[name] = {"ms_per_call": round(tot / args.steps, 4), "launches_per_call": cnt // args.steps}
    T = tc.tc_count_exact(g)["triangles"]
    E2 = 2 * info["m"]
    sweeps = (k + 63) // 64
    model = sweeps * (2 * 8 * E2 + 2 * 4 * 64 * info["n"]) + info["n"] * k // 8
    gbs = model / (ms / 1e3) / 1e9
    print(json.dumps({"metric": "random-projection trace time (1 MI355X) at R-MAT s24, k=256", "value": round(ms, 3),
                      "unit": "ms", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "higher_is_better": False,
                      "dtype": "int64", "data": "synthetic", "estimate": est, "exact": T, "rel_error": est / T - 1.0,
                      "kernels": kern, "model_bytes": model, "roofline": {"bound": "hbm", "achieved": round(gbs, 1),
                      "peak": HBM_PEAK_GBS, "unit": "GB/s", "frac": round(gbs / HBM_PEAK_GBS, 4), "traffic": None},
                      "config": {"workload": "rmat24", "n": info["n"], "m": info["m"], "k": k, "seed": args.seed}}),
          flush=True)


def stream_workload(args):
    """Semi-streaming three-pass estimate (section 5.2) on R-MAT scale 22 with
    d = 1 and 2^24 pass-2 draws: time per call, draws per second, every
    kernel's time, the estimate against the exact count, and parity of the
    seed-0 and seed-1 results with the oracle's stored values.  Roofline of
    the draws' kernel (passes 2 and 3): per draw its number (4 B) and the
    prefix entry, the row offset and the list entry that name its element (16
    B), per lookup a row offset and a list entry (8 B)."""
    import torch
    import synth
    import paper_1011_0468_amd as tc
    n, s, d = synth.workload("rmat22")
    g = tc.tc_build_csr(n, torch.from_numpy(s).cuda(), torch.from_numpy(d).cuda())
    del s, d
    info = g.info()
    S, dd = 1 << 24, 1.0
    golden = _load_golden("stream22.json")
    parity = None
    if golden:
        parity = all(tc.tc_stream_estimate(g, dd, S, seed=r["seed"]) ==
                     {k: r[k] for k in ("draws1", "candidates", "heavy", "light_size", "size", "queries", "closed",
                                        "m", "estimate")} for r in golden["runs"])
    for _ in range(args.warmup):
        tc.tc_stream_estimate(g, dd, S, seed=args.seed)
    tc.profile.select([])
    tc.profile.reset()
    tc.profile.enable(True)
    torch.cuda.synchronize()
    t = time.perf_counter()
    for _ in range(args.steps):
        r = tc.tc_stream_estimate(g, dd, S, seed=args.seed)
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t) * 1e3 / args.steps
    tc.profile.enable(False)
    kern = {}
    for name in ("stream_up", "stream_index", "stream_pass1", "stream_classify", "stream_hlist", "part_count",
                 "part_place", "stream_draws"):
        tot, cnt = tc.profile.read(name)
        if cnt:
            kern[name] = {"ms_per_call": round(tot / args.steps, 4), "launches_per_call": cnt // args.steps}
    m = info["m"]
    draw_bytes = 20 * S + 8 * r["queries"]
    draw_ms = kern.get("stream_draws", {}).get("ms_per_call", 0.0)
    gbs = draw_bytes / (draw_ms / 1e3) / 1e9 if draw_ms else 0.0
    exact = golden["exact"] if golden else None
    print(json.dumps({"metric": "semi-streaming estimate, pass-2 draws/sec at R-MAT s22 (d = 1, 2^24 draws)",
                      "value": round(S / (ms / 1e3), 1), "unit": "draws/s", "n_gpus": 1, "steps": args.steps,
                      "warmup": args.warmup, "ms_per_call": round(ms, 4), "higher_is_better": True,
                      "dtype": "int64", "data": "synthetic", "result": r, "exact": exact,
                      "rel_error": (r["estimate"] / exact - 1.0) if exact else None, "parity_vs_oracle": parity,
                      "kernels": kern,
                      "roofline": {"bound": "hbm", "achieved": round(gbs, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                                   "frac": round(gbs / HBM_PEAK_GBS, 4),
                                   "traffic": _traffic("stream_draws", "rmat22", None, STREAM_SOURCES),
                                   "kernel": "stream_draws", "model_bytes_per_launch": draw_bytes},
                      "config": {"workload": "stream_rmat22", "n": info["n"], "m": m, "d": dd, "num_samples": S,
                                 "seed": args.seed}}), flush=True)


def copy_probe(mib):
    """A plain device copy of known size, for scaling rocprofv3 byte counters."""
    import torch
    a = torch.ones(mib * (1 << 20) // 4, dtype=torch.int32, device="cuda")
    b = torch.empty_like(a)
    for _ in range(3):
        b.copy_(a)
    torch.cuda.synchronize()
    print(json.dumps({"copy_probe_bytes": a.numel() * 4, "launches": 3}))


def main():
    ap = argparse.ArgumentParser(description=__doc__.split("\n")[0])
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=5)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--workload", default="rmat22")
    ap.add_argument("--ps", default="1,0.5,0.1,0.05")
    ap.add_argument("--seed", type=int, default=0)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--copy-probe-mib", type=int, default=0)
    ap.add_argument("--requests", type=int, default=1000, help="serving workload: number of requests")
    ap.add_argument("--serve-requests", type=int, default=100,
                    help="default workload: requests of the short serving trace whose p50/p99 the line reports "
                         "(0: none)")
    ap.add_argument("--pageable", action="store_true",
                    help="serving workload: keep request payloads in pageable host memory")
    ap.add_argument("--tunings", default=None,
                    help="JSON object p -> tuning (the bench line's own 'tunings'): use these instead of autotuning")
    ap.add_argument("--defaults", action="store_true",
                    help="use the library defaults (heavy iff deg > sqrt(m'), default launch parameters) instead of "
                         "the autotuner's choice per operating point")
    args = ap.parse_args()

    world = int(os.environ.get("WORLD_SIZE", "1"))
    if args.gpus != 1 or world != 1:
        print("bench.py runs on exactly one GPU: the counting path has no multi-GPU mode "
              "(--gpus %d, WORLD_SIZE %d requested)" % (args.gpus, world), file=sys.stderr)
        sys.exit(2)

    import torch
    if args.copy_probe_mib:
        copy_probe(args.copy_probe_mib)
        return

    if args.workload == "cl20":
        batched(args)
        return
    if args.workload == "serve":
        serve(args)
        return
    if args.workload == "adaptive":
        adaptive(args)
        return
    if args.workload == "triples":
        triples(args)
        return
    if args.workload == "heavy":
        heavy_stress(args)
        return
    if args.workload == "cl16k":
        latency_cl16k(args)
        return
    if args.workload == "stream":
        stream_workload(args)
        return
    if args.workload == "rp":
        rp_workload(args)
        return

    import synth
    import paper_1011_0468_amd as tc

    ps = [float(x) for x in args.ps.split(",")]
    n, s, d = synth.workload(args.workload)
    src = torch.from_numpy(s).cuda()
    dst = torch.from_numpy(d).cuda()
    torch.cuda.synchronize()
    t = time.perf_counter()
    g = tc.tc_build_csr(n, src, dst)
    torch.cuda.synchronize()
    csr_ms = (time.perf_counter() - t) * 1e3
    del src, dst
    info = g.info()

    tuned = not args.defaults
    given = json.loads(args.tunings) if args.tunings else None
    tunings = {}
    for p in ps:
        if tuned and given is not None:  # a previous run's choice (profiling runs reuse it)
            t = given[str(p)]
            tc.tc_tune_set(g, p, heavy=(t["heavy_num"], t["heavy_den"]), small_dmax=t["small_dmax"],
                           vmajor_cap=t["vmajor_cap"], blocks_per_cu=t["blocks_per_cu"])
            tunings[str(p)] = tc.tc_tune_get(g, p)
        elif tuned:  # untimed, on another sample (seed + 1): launch parameters and heavy multiplier per point
            tunings[str(p)] = tc.tc_autotune(g, p, seed=args.seed + 1, search_heavy=True)
        else:
            tunings[str(p)] = tc.tc_tune_get(g, p)

    def step():
        out = []
        for p in ps:
            if p == 1.0:
                c = tc.tc_count_exact(g, tuned=tuned)
                c["est"] = float(c["triangles"])
            else:
                per, ests, _ = tc.tc_estimate(g, p, [args.seed], tuned=tuned)
                c = per[0]
                c["est"] = ests[0]
            c["p"] = p
            out.append(c)
        return out

    for _ in range(args.warmup):
        step()
    # per-call breakdown (untimed): wall time of each operating point
    per_call_ms = []
    for p in ps:
        torch.cuda.synchronize()
        t = time.perf_counter()
        if p == 1.0:
            tc.tc_count_exact(g, tuned=tuned)
        else:
            tc.tc_estimate(g, p, [args.seed], tuned=tuned)
        torch.cuda.synchronize()
        per_call_ms.append(round((time.perf_counter() - t) * 1e3, 3))

    tc.profile.select([k for names in LIGHT_KERNELS.values() for k in names])
    tc.profile.reset()
    tc.profile.enable(True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        res = step()
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    tc.profile.enable(False)
    ms_per_step = (t1 - t0) * 1e3 / args.steps
    edges = sum(c["m"] for c in res)
    value = edges / (ms_per_step / 1e3)

    # roofline of the dominant kernels: algorithmic bytes / measured launch time
    kern = {}
    for group, names in LIGHT_KERNELS.items():
        reads = [tc.profile.read(k) for k in names]
        model = sum(_light_model_bytes(c, group == "light_large") for c in res) * args.steps
        kern[group] = (sum(r[0] for r in reads), sum(r[1] for r in reads), model)
    dom = max(kern, key=lambda k: kern[k][0])
    ms_tot, launches, model = kern[dom]
    traffic = _traffic(dom, args.workload, tunings)
    # bytes moved where a counter run of these sources is committed, the model's otherwise
    moved = traffic * launches if traffic else model
    achieved = (moved / (ms_tot / 1e3)) / 1e9 if ms_tot > 0 else 0.0
    wedge_bytes = 4 * sum(c["wedges"] for c in res)
    all_light_model = sum(c["model_bytes_small"] + c["model_bytes_large"] for c in res)
    roofline = {"bound": "hbm", "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                "frac": round(achieved / HBM_PEAK_GBS, 4), "traffic": traffic, "kernel": "+".join(LIGHT_KERNELS[dom]),
                "avg_launch_ms": round(ms_tot / max(launches, 1), 4), "launches": launches,
                "basis": "measured traffic" if traffic else "model",
                "model_bytes_per_launch": int(model / max(launches, 1)),
                "model": "list bytes of the light closure (per work item the anchor's list and row offsets, "
                         "per iterated entry 8 B, per probe 4 B; light_bits reads 2 B of them)"}

    phases, phase_ms = phase_breakdown(tc, step, res, info, csr_ms, pairs=len(s))
    line = {
        "metric": "sampled-graph edges/sec (1 MI355X) at R-MAT s22",
        "value": value,
        "unit": "edges/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms_per_step, 4),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "int32",
        "data": "synthetic",
        "config": {"workload": args.workload, "n": info["n"], "m": info["m"], "ps": ps, "seed": args.seed,
                   "split": ("light iff deg <= c sqrt(m'), c = heavy_num/heavy_den per point from the autotuner"
                             if tuned else "light iff deg <= sqrt(m')"),
                   "csr": "int32, resident in HBM"},
        "roofline": roofline,
        "light_wedge_model": {"bytes_per_step": wedge_bytes, "list_bytes_per_step": all_light_model,
                              "note": "the method's lower bound: one 4-byte probe per light wedge"},
        "phases": phases,
        "csr_build_ms": round(csr_ms, 2),
        "per_call_ms": dict(zip([str(p) for p in ps], per_call_ms)),
        "tunings": tunings,
        "results": [{k: c[k] for k in ("p", "m", "triangles", "light", "heavy", "n_heavy", "est")} for c in res],
    }
    line["parity"] = golden_parity(args.workload, args.seed, res, tunings if tuned else None)
    if args.serve_requests > 0:
        sv = serving_trace(args.serve_requests, loads=(0.8,), log=False)
        head = sv["loads"]["0.8"]
        line["serving"] = {"requests": sv["requests"], "load": "0.8 x one-at-a-time capacity",
                           "p50_ms": head["fused"]["p50_ms"], "p99_ms": head["fused"]["p99_ms"],
                           "lanes4_p50_ms": head["lanes4"]["p50_ms"], "lanes4_p99_ms": head["lanes4"]["p99_ms"],
                           "fifo_p50_ms": head["fifo"]["p50_ms"], "fifo_p99_ms": head["fifo"]["p99_ms"],
                           "req_per_s": head["fused"]["req_per_s"], "edges_per_s": head["fused"]["edges_per_s"],
                           "fuse_max_pairs": FUSE_PAIRS,
                           "capacity_req_per_s": sv["capacity_req_per_s"],
                           "identical_alone_and_in_mix": True,
                           "trace": "R-MAT scale uniform in [10, 20], p in {1, .5, .1}, Poisson arrivals seed 12345"}
    if not args.no_cpu_baseline:
        low = [p for p in ps if p <= 0.1]
        gms = {p: per_call_ms[ps.index(p)] for p in low}
        cb, counts = cpu_baseline(args.workload, low, [args.seed, args.seed + 1, args.seed + 2], gms)
        gc = {c["p"]: c["triangles"] for c in res}
        cb["parity_with_gpu"] = all(counts[(p, args.seed)]["triangles"] == gc[p] for p in low)
        line["cpu_baseline"] = cb
    print(json.dumps(line), flush=True)


def _mfma_ops(h):
    """int8 MFMA operations the heavy kernel executes for h heavy vertices:
    2 * 128^3 * (J - I + 1) per 128 x 128 macro tile I <= J."""
    nm = (h + 127) // 128
    return 2 * 128 ** 3 * sum((J + 1) * (J + 2) // 2 for J in range(nm)) if h >= 3 else 0


def phase_breakdown(tc, step, res, info, csr_ms, pairs):
    """One extra step with every launch bracketed by HIP events (outside the
    timed region): kernel time per step of the path, next to the bytes or
    operations its model says it must move (the declared per-phase models:
    sample 4*2m + 4(n+1) read + 4*2m' + 8(n+1) written; orientation and split
    4*2m' + 4(n+1) read + 4m' + 4(n+1) + 4n written; light closure: the list
    model; heavy block: executed int8 MFMA operations; CSR build 8 B per input
    pair read, 4*2m + 8n + 4 written)."""
    import torch
    tc.profile.select([])
    tc.profile.reset()
    tc.profile.enable(True)
    torch.cuda.synchronize()
    t = time.perf_counter()
    step()
    torch.cuda.synchronize()
    wall = (time.perf_counter() - t) * 1e3
    tc.profile.enable(False)
    ms = {ph: tc.profile.read("@" + ph)[0] for ph in ("sample", "orient", "light", "heavy", "finish")}
    n, m = info["n"], info["m"]
    sampled = [c for c in res if c["p"] < 1.0]
    b_sample = sum(4 * 2 * m + 4 * (n + 1) + 4 * 2 * c["m"] + 8 * (n + 1) for c in sampled)
    b_orient = sum(4 * 2 * c["m"] + 4 * (n + 1) + 4 * c["m"] + 4 * (n + 1) + 4 * n for c in res)
    b_light = sum(c["model_bytes_small"] + c["model_bytes_large"] for c in res)
    ops_heavy = sum(_mfma_ops(c["n_heavy"]) for c in res)
    b_csr = 8 * pairs + 4 * 2 * m + 8 * n + 4

    def hbm(b, t_ms):
        gbs = b / (t_ms / 1e3) / 1e9 if t_ms > 0 else 0.0
        return {"ms": round(t_ms, 4), "model_bytes": int(b), "gbs": round(gbs, 1), "frac": round(gbs / HBM_PEAK_GBS, 4)}

    out = {"sample": hbm(b_sample, ms["sample"]), "orient_split": hbm(b_orient, ms["orient"]),
           "light": hbm(b_light, ms["light"]),
           "heavy": {"ms": round(ms["heavy"], 4), "mfma_ops": ops_heavy,
                     "tops": round(ops_heavy / (ms["heavy"] / 1e3) / 1e12, 2) if ms["heavy"] > 0 else 0.0,
                     "frac_int8_peak": round(ops_heavy / (ms["heavy"] / 1e3) / 1e12 / 5000.0, 5)
                     if ms["heavy"] > 0 else 0.0},
           "finish_ms": round(ms["finish"], 4),
           "kernel_ms_sum": round(sum(ms.values()), 4), "step_wall_ms": round(wall, 4),
           "csr_build": hbm(b_csr, csr_ms)}
    out["light"]["wedge_bound_bytes"] = 4 * sum(c["wedges"] for c in res)
    out["light"]["frac_wedge_bound"] = round(out["light"]["wedge_bound_bytes"] / (ms["light"] / 1e3) / 1e9
                                             / HBM_PEAK_GBS, 4) if ms["light"] > 0 else 0.0
    out["note"] = ("kernel time from HIP events around every launch of one untimed step; the csr_build time is "
                   "the wall time of tc_build_csr")
    return out, ms


def _load_golden(name):
    """A stored oracle result under tests/golden (None if absent)."""
    try:
        return json.load(open(os.path.join(ROOT, "tests", "golden", name)))
    except (OSError, ValueError):
        return None


def golden_parity(workload, seed, res, tunings):
    """The step's counts against the oracle's stored values (tests/golden,
    written by tests/golden/make_golden.py from the oracle alone): per point
    the triangle count, and the light/heavy split for the multiplier used."""
    if workload != "rmat22" or seed != 0:
        return None
    gd = os.path.join(ROOT, "tests", "golden")
    want = {}
    try:
        for c in json.load(open(os.path.join(gd, "rmat22.json")))["counts"]:
            want[(c["p"], 1, 1)] = c
        if os.path.exists(os.path.join(gd, "rmat22_splits.json")):
            for c in json.load(open(os.path.join(gd, "rmat22_splits.json")))["counts"]:
                want[(c["p"], c["split"][0], c["split"][1])] = c
    except (OSError, ValueError, KeyError):
        return None
    out = {}
    for c in res:
        t = tunings[str(c["p"])] if tunings else {"heavy_num": 1, "heavy_den": 1}
        a, b = t["heavy_num"], t["heavy_den"]
        import math
        gcd = math.gcd(a, b) or 1
        w = want.get((c["p"], a // gcd, b // gcd))
        if w is None:
            out[str(c["p"])] = "no stored split for c = %d/%d" % (a, b)
            continue
        ok = all(c[k] == w[k] for k in ("triangles", "light", "heavy", "n_heavy", "m"))
        out[str(c["p"])] = "equal" if ok else "DIFFERENT"
    return out


if __name__ == "__main__":
    main()
