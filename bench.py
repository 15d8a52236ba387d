#!/usr/bin/env python3
"""Benchmark: BFS + SSSP from 64 sources on an R-MAT scale-22 graph.

Workload (one "step"): a BFS and an SSSP from each of 64 sources drawn
uniformly from the largest component of a seeded R-MAT graph (scale 22, edge
factor 16, (a,b,c,d) = (0.57,0.19,0.19,0.05), symmetrised, simple, int32 CSR,
uint32 weights uniform in [1,64]).  Inputs are synthetic and resident in HBM
before timing; outputs (64 x n depths and 64 x n distances) are written to
device buffers.

value = GTEPS over the step: for every solve, the sum of the degrees of the
vertices it reaches (the paper's directed-edge convention), summed over all
128 solves and divided by the step time.

The JSON line also carries:
  roofline      the dominant kernel's algorithmic bytes per launch / its
                average launch time (HIP events on the launch stream, in a
                second pass over the same steps), against 8 TB/s HBM peak
  cpu_baseline  the CPU oracle (1 thread) on a bounded sample of the work
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0


def kernel_source_digest(files=None) -> str:
    """Hash of the engine sources (all of csrc/ by default, else the named
    files, paths relative to the package)."""
    pkg = os.path.join(ROOT, "paper_1501_05387_amd")
    if files is None:
        files = ["csrc/" + f for f in sorted(os.listdir(os.path.join(pkg, "csrc")))]
    h = hashlib.sha256()
    for f in files:
        h.update(os.path.basename(f).encode())
        h.update(open(os.path.join(pkg, f), "rb").read())
    return h.hexdigest()[:16]


# Everything the batched relaxation kernel is compiled from: its source file,
# the headers it includes and the build flags.  A counter figure taken for
# that kernel stays valid while these are unchanged.
RELAX_SOURCES = ["csrc/sssp_batch.hip", "csrc/compact.h", "csrc/device.h", "csrc/engine.h", "csrc/entries.h",
                 "csrc/batches.h", "csrc/error.h", "csrc/nearness.h", "csrc/spare.h", "../include/gfr.h", "build.py"]


def relax_source_digest() -> str:
    return kernel_source_digest(RELAX_SOURCES)


def bfs_bytes(st: dict, solves: int, n: int) -> float:
    """Algorithmic bytes of bfs_level over `solves` BFS (traffic model of the design notes)."""
    push = 12 * st["push_entries"] + 8 * st["push_edges"] + 16 * st["push_new"]
    pull = (n / 4.0) * st["pull_levels"] + 8 * st["pull_unvisited"] + 8 * st["pull_inspected"] \
        + 16 * st["pull_new"]
    return push + pull


def bsssp_bytes(st: dict) -> float:
    """Algorithmic bytes of bsssp_relax over its queries, by the SSSP work model:
    16 B per (vertex, query) frontier entry (queue slot and distance), 12 B per
    (edge, query) relaxation (column, weight, target distance) and 8 B per
    improvement (the atomic update and its mark).  These are the method's own
    bytes, the same per query as for a single-source solve; the batched kernel
    shares every column and weight among the queries active on an edge."""
    return 16 * st["pair_entries"] + 12 * st["lane_relaxations"] + 8 * st["improvements"]


def bsssp_floor_bytes(pairs: int, edges: int, queries: int) -> float:
    """The SSSP work model at its floor (re-relaxation factor r = 1): every
    reached (vertex, query) pair enters the frontier once (16 B), every edge
    leaving it is relaxed once for that query (12 B) and every reached pair
    other than a source is improved once (8 B).  Fixed by the solves' results
    alone, so no schedule, re-relaxation or speculative relaxation is credited
    with bytes."""
    return 16 * pairs + 12 * edges + 8 * (pairs - queries)


def bsssp_row_bytes(st: dict) -> float:
    """Bytes the batched layout moves per edge visit: column and weight (8 B)
    plus the target's whole 64-query distance row (256 B), plus 4 B per
    improvement.  A layout figure (what the kernel touches), not the work
    model."""
    return (8 + 256) * st["relaxations"] + 4 * st["improvements"]


def host_cpu() -> tuple:
    """(logical cores, CPU model name) of this host."""
    model = "unknown"
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                model = line.split(":", 1)[1].strip()
                break
    except OSError:
        pass
    return os.cpu_count() or 0, model


def msbfs_bytes(st: dict, n: int) -> float:
    """Algorithmic bytes of msbfs_level: push edges read column + visited and
    next masks (20 B); a pull level reads every row offset and visited mask
    (12 B per vertex) plus, per inspected edge, column and frontier mask (12 B),
    bounded here by one full sweep of the edges."""
    m_edges = st.get("m", 0)
    return 20 * st.get("push_edges", 0) + st.get("pull_levels", 0) * (12 * n + 12 * m_edges)


def sssp_bytes(st: dict) -> float:
    """Algorithmic bytes of sssp_relax: per near entry its queue slot and distance (16 B),
    per relaxed edge column, weight and target distance (12 B), per improvement one
    atomic read-modify-write of the distance and one mark (8 B)."""
    return 16 * st["near_entries"] + 12 * st["relaxations"] + 8 * st["improvements"]


STAT_KEYS = ["m", "push_entries", "push_edges", "push_new", "pull_levels", "pull_unvisited",
             "pull_inspected", "pull_new", "near_entries", "relaxations", "lane_relaxations",
             "pair_entries", "improvements", "far_entries", "iterations", "levels", "launches", "solves"]


def read_stats(ctx, keys):
    out = {}
    for k in keys:
        try:
            out[k] = ctx.stat(k)
        except Exception:
            pass
    return out


SERVE_SCALES = (18, 19, 20, 21, 22, 23)
SERVE_RATES = (500.0, 2000.0, 8000.0, 1e9)


def serve_leg(ctx, resident, nq, log, rates=SERVE_RATES, modes=("batched", "one_at_a_time")):
    """The serving workload: six resident R-MAT graphs (scales 18-23, edge
    factor 16, weights in [1,64]); a Poisson stream of queries, 70 % BFS and
    30 % SSSP, each on a graph drawn Zipf(s = 1.2) over the scales in
    ascending order (scale 18 the most popular) from a random source of that
    graph's largest component; a ladder of offered rates.  Served batched
    (continuous batching, up to 64 queries per session) and one at a time
    (single-source solvers), on the same GPU, with every result checked
    against the same query solved directly."""
    import torch

    import graphgen
    import paper_1501_05387_amd as gfr
    rng = np.random.default_rng(graphgen.SEED_ARRIVALS)
    zipf = np.array([1.0 / (i + 1) ** 1.2 for i in range(len(SERVE_SCALES))])
    zipf /= zipf.sum()
    pools = {s: graphgen.sample_sources(r, c, 256, seed=graphgen.SEED_ARRIVALS) for s, (r, c, _, _) in resident.items()}
    gsel = rng.choice(len(SERVE_SCALES), size=nq, p=zipf)
    scales = [SERVE_SCALES[i] for i in gsel]
    srcs = [int(pools[s][rng.integers(0, pools[s].size)]) for s in scales]
    kinds = np.where(rng.random(nq) < 0.7, gfr.GFR_Q_BFS, gfr.GFR_Q_SSSP)
    outs = [torch.empty(resident[s][0].size - 1, dtype=torch.int32, device="cuda:0") for s in scales]
    # reference results, each query solved directly
    ref = {}
    for i in range(nq):
        key = (scales[i], int(kinds[i]), srcs[i])
        if key not in ref:
            g = resident[scales[i]][3]
            ref[key] = (ctx.bfs(g, srcs[i]) if kinds[i] == gfr.GFR_Q_BFS else ctx.sssp(g, srcs[i])).clone()
    res = {}
    for mode, mb in (("batched", 64), ("one_at_a_time", 1)):
        if mode not in modes:
            continue
        ctx.set_option("serve.max_batch", mb)
        pts = []
        for rate in rates:
            gaps = rng.exponential(1.0 / rate, size=nq)
            arrive = np.cumsum(gaps) - gaps[0]
            for o in outs:
                o.fill_(-7)
            torch.cuda.synchronize()
            ctx.stat("serve.reset")
            done = {}
            t_sub = np.zeros(nq)
            t_end = {}
            tick_of = {}

            def drain(timeout_us):
                got = ctx.poll(256, timeout_us)
                now = time.perf_counter()
                for t, st in got:
                    done[t] = st
                    t_end[t] = now

            t0 = time.perf_counter()
            for i in range(nq):
                while time.perf_counter() - t0 < arrive[i]:
                    drain(0)
                t_sub[i] = time.perf_counter()
                tick_of[ctx.submit_queries([(int(kinds[i]), resident[scales[i]][3], srcs[i], outs[i])])[0]] = i
            while len(done) < nq:
                drain(100000)
            span = time.perf_counter() - t0
            ok = all(st == gfr.GFR_OK for st in done.values()) and all(
                torch.equal(outs[i], ref[(scales[i], int(kinds[i]), srcs[i])]) for i in range(nq))
            # per-query latency seen by the caller (submit -> poll returns it), by class
            lat = np.zeros(nq)
            for t, i in tick_of.items():
                lat[i] = (t_end[t] - t_sub[i]) * 1e3
            p99 = float(np.percentile(lat, 99))
            cls = {}
            for sc in SERVE_SCALES:
                for kd, kn in ((gfr.GFR_Q_BFS, "bfs"), (gfr.GFR_Q_SSSP, "sssp")):
                    sel = np.array([scales[i] == sc and kinds[i] == kd for i in range(nq)])
                    if sel.any():
                        cls["s%d_%s" % (sc, kn)] = {"n": int(sel.sum()),
                                                   "p50_ms": round(float(np.percentile(lat[sel], 50)), 3),
                                                   "p99_ms": round(float(np.percentile(lat[sel], 99)), 3),
                                                   "in_tail": int((lat[sel] > p99).sum())}
            pts.append({"offered_qps": rate if rate < 1e8 else None, "qps": round(nq / span, 1),
                        "p50_ms": round(ctx.stat("serve.p50_ms"), 3), "p99_ms": round(ctx.stat("serve.p99_ms"), 3),
                        "caller_p50_ms": round(float(np.percentile(lat, 50)), 3), "caller_p99_ms": round(p99, 3),
                        "mean_batch": round(ctx.stat("serve.mean_batch"), 2),
                        "joined_running": int(ctx.stat("serve.joined")), "results_equal": bool(ok),
                        "by_class": cls})
            log("serve %s rate %s: %s" % (mode, rate, {k: v for k, v in pts[-1].items() if k != "by_class"}))
        res[mode] = pts
    ctx.set_option("serve.max_batch", 64)
    res["queries_per_point"] = nq
    res["mix"] = ("6 R-MAT graphs s18-s23 resident; 70% BFS / 30% SSSP; graph Zipf(1.2) over ascending scales; "
                  "sources from each graph's largest component; Poisson arrivals")
    return res


def main():
    ap = argparse.ArgumentParser(description=__doc__, formatter_class=argparse.RawDescriptionHelpFormatter)
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=3)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--scale", type=int, default=22)
    ap.add_argument("--edge-factor", type=int, default=16)
    ap.add_argument("--sources", type=int, default=64)
    ap.add_argument("--cpu-sources", type=int, default=5, help="oracle sample size (sources, about 12 s of CPU work)")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--serve-queries", type=int, default=10000, help="queries per serving point (0: skip)")
    ap.add_argument("--serve-rates", default="500,2000,8000,burst",
                    help="offered rates of the serving points, queries/s ('burst': all at once)")
    ap.add_argument("--serve-modes", default="batched,one_at_a_time", help="serving modes to run")
    ap.add_argument("--copy-probe-mib", type=int, default=0,
                    help="finish with one device copy of this many MiB (a known-size kernel that "
                         "calibrates the HBM byte counters of a profiler run)")
    args = ap.parse_args()

    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py: the engine runs on one GPU only (it is single-device); "
              "use --gpus 1", file=sys.stderr)
        sys.exit(2)

    import torch

    import graphgen
    import paper_1501_05387_amd as gfr

    def log(*a):
        print("[bench]", *a, file=sys.stderr, flush=True)

    t0 = time.time()
    row, col = graphgen.rmat(args.scale, args.edge_factor)
    w = graphgen.weights(row, col, 64)
    srcs = graphgen.sample_sources(row, col, args.sources)
    n, m = row.size - 1, col.size
    log("graph scale %d: n=%d m=%d (%.1fs)" % (args.scale, n, m, time.time() - t0))

    ctx = gfr.Context(0, tuning_json=gfr.tuned_json())   # the autotuner's per-class choices (results-neutral)
    g = ctx.graph_load_csr(row, col, w)
    dev = torch.device("cuda:0")
    dep = torch.empty(args.sources * n, dtype=torch.int32, device=dev)
    dist = torch.empty(args.sources * n, dtype=torch.int32, device=dev)

    def step():
        ctx.bfs_batch(g, srcs, out=dep)
        ctx.sssp_batch(g, srcs, out=dist)

    # the warm-up runs with the per-launch events on as well, so that the
    # library's event pool exists before the timed steps; events bracket the
    # advance kernels only (every launch bracketed would cost the step 0.8 ms)
    ctx.set_option("profile.kernels", 2)
    for i in range(args.warmup):
        step()
        log("warmup step %d done" % i)
    torch.cuda.synchronize()

    # edges traversed per step: each solve counts the degrees of the vertices it reaches
    deg = torch.from_numpy(np.diff(row).astype(np.int64)).to(dev)
    d2 = dep.view(args.sources, n)
    te_bfs = sum(int(deg[d2[i] >= 0].sum().item()) for i in range(args.sources))
    s2 = dist.view(args.sources, n)
    te_sssp = sum(int(deg[s2[i] != -1].sum().item()) for i in range(args.sources))
    pairs_sssp = int((s2 != -1).sum().item())   # reached (vertex, query) pairs, sources included

    # timed steps; HIP events on the library's launch stream bracket every level
    # kernel inside them (profile.kernels), which gives the roofline figures
    # of the same launches that the step time covers
    knames = ("msbfs_level", "bsssp_relax")
    kacc = {k: [0.0, 0.0] for k in knames}
    sb_acc, ss_acc = {}, {}

    def kstat(name):
        try:
            return ctx.stat("t.%s.ms" % name), ctx.stat("t.%s.n" % name)
        except Exception:
            return 0.0, 0.0

    def add(acc, st):
        for key, v in st.items():
            acc[key] = acc.get(key, 0.0) + v

    read_stats(ctx, STAT_KEYS)   # the first statistics query of a process is slow (~80 ms); keep it untimed
    for k in knames:
        kstat(k)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    for i in range(args.steps):
        ctx.bfs_batch(g, srcs, out=dep)
        add(sb_acc, read_stats(ctx, STAT_KEYS))
        for k in knames[:1]:
            ms_, n_ = kstat(k)
            kacc[k][0] += ms_
            kacc[k][1] += n_
        ctx.sssp_batch(g, srcs, out=dist)
        add(ss_acc, read_stats(ctx, STAT_KEYS))
        for k in knames[1:]:
            ms_, n_ = kstat(k)
            kacc[k][0] += ms_
            kacc[k][1] += n_
    torch.cuda.synchronize()
    t_step = (time.perf_counter() - t1) / args.steps
    ctx.set_option("profile.kernels", 0)
    value = (te_bfs + te_sssp) / t_step / 1e9
    log("timed %d steps: %.2f ms/step, %.1f GTEPS" % (args.steps, t_step * 1e3, value))

    # the same step with host output buffers (results cross PCIe inside the calls)
    hdep = np.empty(args.sources * n, np.int32)
    hdist = np.empty(args.sources * n, np.uint32)
    torch.cuda.synchronize()
    th = time.perf_counter()
    ctx.bfs_batch(g, srcs, out=hdep)
    ctx.sssp_batch(g, srcs, out=hdist)
    t_host = time.perf_counter() - th
    host_ok = bool(np.array_equal(hdep, dep.cpu().numpy()) and np.array_equal(hdist.view(np.int32), dist.cpu().numpy()))
    log("host-output step: %.2f ms (%.1f GTEPS incl. PCIe), same results %s"
        % (t_host * 1e3, (te_bfs + te_sssp) / t_host / 1e9, host_ok))
    del hdep, hdist

    # per-primitive split of one step (library event timing of each whole call)
    torch.cuda.synchronize()
    ctx.bfs_batch(g, srcs, out=dep)
    ms_bfs = ctx.stat("kernel_ms")
    ctx.sssp_batch(g, srcs, out=dist)
    ms_sssp = ctx.stat("kernel_ms")

    # roofline of the dominant kernel over the timed steps (K steps of work)
    sb = dict(sb_acc, m=m)   # counts summed over the steps; m is the graph's
    ss = ss_acc
    ktimes = {k: tuple(v) for k, v in kacc.items()}
    kernels = {k: {"ms": v[0], "launches": v[1]} for k, v in ktimes.items()}
    kernels["bsssp_relax"]["bytes"] = bsssp_floor_bytes(pairs_sssp, te_sssp, args.sources) * args.steps
    kernels["bsssp_relax"]["counted_bytes"] = bsssp_bytes(ss)
    kernels["bsssp_relax"]["row_layout_bytes"] = bsssp_row_bytes(ss)
    kernels["msbfs_level"]["bytes"] = msbfs_bytes(sb, n)
    for k in ("bsssp_relax", "msbfs_level"):
        kernels[k]["GBs"] = kernels[k]["bytes"] / max(kernels[k]["ms"], 1e-9) / 1e6
    dom = max(("msbfs_level", "bsssp_relax"), key=lambda k: kernels[k]["ms"])
    kd = kernels[dom]
    achieved = kd["bytes"] / kd["launches"] / (kd["ms"] / kd["launches"] * 1e-3) / 1e9
    # measured HBM bytes per launch: not counted by this run (a counter run
    # is a profiler pass of its own); taken from the committed counter
    # summary when it was made for the current kernel sources, else null
    traffic, traffic_src = None, None
    tfile = os.path.join(ROOT, "profiles", "traffic.json")
    if os.path.exists(tfile):
        tj = json.load(open(tfile))
        ent = tj.get("%s/rmat%d" % (dom, args.scale))
        want = relax_source_digest() if dom == "bsssp_relax" else kernel_source_digest()
        if ent and ent.get("source_digest") == want:
            traffic = ent.get("bytes_per_launch")
            traffic_src = "copied from profiles/traffic.json (rocprofv3 FETCH_SIZE + WRITE_SIZE, same kernel sources)"
    roofline = {"bound": "hbm", "kernel": dom, "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS,
                "unit": "GB/s", "frac": round(achieved / HBM_PEAK_GBS, 4), "traffic": traffic,
                "traffic_source": traffic_src,
                "bytes_per_launch": kd["bytes"] / kd["launches"],
                "bytes_model": ("SSSP work model at r = 1: 16 B per reached (vertex, query) pair + 12 B per "
                                "(edge, query) leaving it + 8 B per improvement, per step over the step's "
                                "launches" if dom == "bsssp_relax" else "see msbfs_bytes"),
                "avg_launch_us": kd["ms"] / kd["launches"] * 1e3}
    if dom == "bsssp_relax":
        # the same model over the entries, relaxations and improvements the
        # kernel counted (re-relaxations and pending-query relaxations
        # included; these share the row visit of the frontier's own lanes, so
        # the figure can exceed the bytes that reach HBM)
        roofline["counted_bytes_per_launch"] = kd["counted_bytes"] / kd["launches"]
        roofline["row_layout_bytes_per_launch"] = kd["row_layout_bytes"] / kd["launches"]
        # re-relaxation factor: (edge, query) relaxations over the edges the
        # queries reach (sum of reached degrees), the floor of one relaxation each
        roofline["r_lane"] = round(ss["lane_relaxations"] / (te_sssp * args.steps), 4)
        roofline["edge_visits_per_batch_over_m"] = round(
            ss["relaxations"] / args.steps / max(1, (args.sources + 63) // 64) / m, 4)
    log("kernels:", json.dumps(kernels))

    cpu = None
    parity = None
    if not args.no_cpu_baseline:
        import oracle
        k = max(1, min(args.cpu_sources, args.sources))
        te = 0
        tc = 0.0
        ok = True
        for i in range(k):
            s = int(srcs[i])
            ta = time.perf_counter()
            db = oracle.bfs(row, col, s)
            ds = oracle.sssp(row, col, w, s)
            tc += time.perf_counter() - ta
            reached = db >= 0
            te += 2 * int(np.diff(row)[reached].sum())
            ok = ok and np.array_equal(d2[i].cpu().numpy(), db)
            ok = ok and np.array_equal(s2[i].cpu().numpy().view(np.uint32), ds)
        ncores, model = host_cpu()
        cpu = {"value": round(te / tc / 1e9, 4), "unit": "GTEPS", "cores": 1, "kind": "oracle",
               "host_cores": ncores, "cpu_model": model,
               "sample": "queue BFS + binary-heap Dijkstra from %d of the %d sources, 1 thread of %d host "
                         "cores (%s), %.1f s" % (k, args.sources, ncores, model, tc)}
        parity = ok
        log("cpu oracle: %.3f GTEPS on %d source(s), parity %s" % (te / tc / 1e9, k, ok))

    serving = None
    if args.serve_queries > 0:
        resident = {}
        for sc in SERVE_SCALES:
            if sc == args.scale and args.edge_factor == 16:
                resident[sc] = (row, col, w, g)
                continue
            r2, c2 = graphgen.rmat(sc, 16)
            w2 = graphgen.weights(r2, c2, 64)
            resident[sc] = (r2, c2, w2, ctx.graph_load_csr(r2, c2, w2))
            log("serving graph scale %d loaded (n=%d m=%d)" % (sc, r2.size - 1, c2.size))
        rates = tuple(1e9 if r.strip() == "burst" else float(r) for r in args.serve_rates.split(","))
        serving = serve_leg(ctx, resident, args.serve_queries, log, rates=rates,
                            modes=tuple(m.strip() for m in args.serve_modes.split(",")))
        log("serving:", json.dumps(serving))
        for sc, (_, _, _, g2) in resident.items():
            if g2 is not g:
                g2.free()

    line = {
        "metric": "BFS/SSSP GTEPS on R-MAT s22 ef16 (HBM GB/s); batched queries/s + p99 latency",
        "value": round(value, 3),
        "unit": "GTEPS",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(t_step * 1e3, 3),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "u32",
        "data": "synthetic",
        "config": {"workload": "rmat%d_ef%d_bfs_sssp_%dsrc" % (args.scale, args.edge_factor, args.sources),
                   "scale": args.scale, "edge_factor": args.edge_factor, "n": n, "m": m,
                   "sources": args.sources, "weights": "uniform[1,64]", "parallelism": "single-gpu"},
        "roofline": roofline,
        "cpu_baseline": cpu,
        "detail": {"gteps_bfs": round(te_bfs / (ms_bfs * 1e-3) / 1e9, 3),
                   "gteps_sssp": round(te_sssp / (ms_sssp * 1e-3) / 1e9, 3),
                   "ms_bfs_64": round(ms_bfs, 3), "ms_sssp_64": round(ms_sssp, 3),
                   "edges_traversed_per_step": te_bfs + te_sssp, "kernels": kernels,
                   "parity_sample_ok": parity, "source_digest": kernel_source_digest(),
                   "serving": serving,
                   "host_output_step_ms": round(t_host * 1e3, 3),
                   "host_output_gteps": round((te_bfs + te_sssp) / t_host / 1e9, 3),
                   "host_output_same": host_ok},
    }
    print(json.dumps(line), flush=True)
    if args.copy_probe_mib > 0:
        # an elementwise kernel (not a DMA copy) that reads and writes exactly nb bytes
        nw = (args.copy_probe_mib << 20) // 4
        a = torch.ones(nw, dtype=torch.int32, device=dev)
        b = torch.empty(nw, dtype=torch.int32, device=dev)
        torch.cuda.synchronize()
        torch.bitwise_not(a, out=b)
        torch.cuda.synchronize()
        log("copy probe: bitwise_not over %d MiB (reads and writes %d bytes)" % (args.copy_probe_mib, nw * 4))
        # a second known-size kernel that only reads: the sum of the same words
        tot = int(torch.sum(a).item())
        log("read probe: sum over %d MiB (reads %d bytes), total %d" % (args.copy_probe_mib, nw * 4, tot))
        del a, b
    g.free()
    ctx.close()


if __name__ == "__main__":
    main()
