"""Performance cases of the frontier graph engine, through its Python entry points.

A case is a plain dict: the call (``op``), the graph it runs on (``graph``,
``n`` or ``side``, ``ef``) and the call's own options.  ``prepare`` makes what a
user's program has in hand before the call: a context with the packaged tuning
file (or the library's defaults), the resident graph, the sources, the caller's
frontier.  ``run`` makes the call.

Graphs are the two kinds that the engine is measured on elsewhere: R-MAT
((0.57, 0.19, 0.19, 0.05), symmetric, simple; ``n`` need not be a power of two,
draws outside are dropped) and the perturbed square lattice (3 % of the edges
dropped, 0.1 % long edges).  They are drawn on the GPU from the seed.
"""
import math

import numpy as np
import torch

import paper_1501_05387_amd as gfr

DEV = "cuda:0"
GIANT = 1 << 62


def listed():
    return [
        # one query on a small resident graph: launches, synchronisation and latency
        {"name": "bfs_rmat_1k", "op": "bfs", "graph": "rmat", "n": 1024, "ef": 16, "pred": False, "host": False,
         "tuned": True},
        # the direction-optimizing traversal of a large scale-free graph
        {"name": "bfs_rmat_4m", "op": "bfs", "graph": "rmat", "n": 1 << 22, "ef": 16, "pred": False, "host": False,
         "tuned": True},
        # long-diameter graph (road network, mesh): about 140 thin levels
        {"name": "bfs_lattice_4096", "op": "bfs", "graph": "lattice", "side": 4096, "pred": False, "host": False,
         "tuned": True},
        # shortest paths with the route back (predecessors), ragged vertex count
        {"name": "sssp_rmat_1m_pred", "op": "sssp", "graph": "rmat", "n": 1000003, "ef": 16, "maxw": 64,
         "pred": True, "host": False, "tuned": True},
        # shortest paths on a mesh, odd side, wide weights: hundreds of thin iterations
        {"name": "sssp_lattice_1999", "op": "sssp", "graph": "lattice", "side": 1999, "maxw": 1000, "pred": False,
         "host": False, "tuned": True},
        # 64 sources that share the traversal (all-pairs samples, landmark tables)
        {"name": "bfs_batch_rmat_1m", "op": "bfs_batch", "graph": "rmat", "n": 1 << 20, "ef": 16, "k": 64,
         "host": False, "tuned": True},
        # the benchmark's shortest-path half, the largest call
        {"name": "sssp_batch_rmat_4m", "op": "sssp_batch", "graph": "rmat", "n": 1 << 22, "ef": 16, "maxw": 64,
         "k": 64, "host": False, "tuned": True},
        # a part-filled batch on an ordinary graph, results wanted in host memory
        {"name": "sssp_batch_rmat_50k_host", "op": "sssp_batch", "graph": "rmat", "n": 50021, "ef": 12, "maxw": 64,
         "k": 21, "host": True, "tuned": True},
        # forward and backward passes over sampled sources
        {"name": "bc_rmat_1m", "op": "bc", "graph": "rmat", "n": 1 << 20, "ef": 16, "k": 4, "tuned": True},
        # components of a mesh: long label chains
        {"name": "cc_lattice_3001", "op": "cc", "graph": "lattice", "side": 3001, "tuned": True},
        # power iteration to convergence on a large scale-free graph
        {"name": "pagerank_rmat_4m", "op": "pagerank", "graph": "rmat", "n": 1 << 22, "ef": 16, "tol": 1e-6,
         "tuned": True},
        # a caller's own traversal step out of the operators: advance, filter, split, scan, into buffers of a fixed
        # number of edges
        {"name": "step_rmat_260k", "op": "step", "graph": "rmat", "n": 260017, "ef": 16, "maxw": 64, "edges": 180001,
         "tuned": True},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# op: largest R-MAT n, largest lattice side (0: not drawn on a lattice)
_DRAW = {"bfs": (1 << 22, 4096), "sssp": (1 << 21, 2048), "bfs_batch": (1 << 20, 1024), "sssp_batch": (1 << 20, 300),
         "bc": (1 << 20, 300), "cc": (1 << 22, 3001), "pagerank": (1 << 22, 2048), "step": (1 << 20, 1024)}


def draw(rng):
    op = rng.choice(sorted(_DRAW))
    big, side = _DRAW[op]
    c = {"op": op, "tuned": rng.random() < 0.75}
    if rng.random() < 0.35:
        c.update(graph="lattice", side=_log(rng, 33, side))
        n = c["side"] ** 2
    else:
        n = _log(rng, 1000, big)
        c.update(graph="rmat", n=n, ef=rng.choice([8, 12, 16]))
    if op in ("sssp", "sssp_batch", "step"):
        c["maxw"] = rng.choice([64, 1000])
    if op in ("bfs", "sssp"):
        c["pred"] = rng.random() < 0.3
    if op in ("bfs", "sssp", "bfs_batch", "sssp_batch"):
        c["host"] = rng.random() < 0.2
    if op in ("bfs_batch", "sssp_batch"):
        c["k"] = rng.randint(2, 64)
    if op == "bc":
        c["k"] = rng.randint(1, 4)
    if op == "pagerank":
        c["tol"] = rng.choice([1e-4, 1e-6])
    if op == "step":
        c["edges"] = _log(rng, 100, n)
    return c


# ---------------------------------------------------------------- inputs
def _vertices(case):
    return case["side"] ** 2 if case["graph"] == "lattice" else case["n"]


def _edges(case):
    """Expected directed entries."""
    if case["graph"] == "lattice":
        return int(4 * case["side"] * (case["side"] - 1) * 0.971)
    return int(2 * case["n"] * case["ef"] * 0.9)


def _rmat_pairs(n, ef, gen):
    scale = max(1, (n - 1).bit_length())
    count = ef * n
    u = torch.zeros(count, dtype=torch.int64, device=DEV)
    v = torch.zeros(count, dtype=torch.int64, device=DEV)
    for _ in range(scale):
        r = torch.rand(count, generator=gen, device=DEV)
        low = r >= 0.76
        u = u * 2 + low
        v = v * 2 + (((r >= 0.57) & ~low) | (r >= 0.95))
    keep = (u < n) & (v < n)
    return u[keep], v[keep]


def _lattice_pairs(side, gen):
    ids = torch.arange(side * side, dtype=torch.int64, device=DEV).view(side, side)
    u = torch.cat([ids[:, :-1].reshape(-1), ids[:-1, :].reshape(-1)])
    v = torch.cat([ids[:, 1:].reshape(-1), ids[1:, :].reshape(-1)])
    keep = torch.rand(u.numel(), generator=gen, device=DEV) >= 0.03
    long = torch.randint(0, side * side, (2, max(1, u.numel() // 1000)), generator=gen, device=DEV)
    return torch.cat([u[keep], long[0]]), torch.cat([v[keep], long[1]])


def _csr(case, seed):
    """Symmetric simple CSR on the GPU: row offsets and columns (int64), and the generator after the draws."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    n = _vertices(case)
    u, v = _lattice_pairs(case["side"], gen) if case["graph"] == "lattice" else _rmat_pairs(n, case["ef"], gen)
    keep = u != v
    u, v = u[keep], v[keep]
    key = torch.unique(torch.cat([u * n + v, v * n + u]))
    u, v = key // n, key % n
    row = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    row[1:] = torch.cumsum(torch.bincount(u, minlength=n), 0)
    return row, u, v, gen


def _weights(u, v, maxw, n, seed):
    """Symmetric integer weights in [1, maxw], a hash of the unordered pair."""
    h = torch.minimum(u, v) * n + torch.maximum(u, v) + (seed % 1000003) * 7919
    h = (h ^ (h >> 29)) * -4658895280553007687
    h = (h ^ (h >> 32)) * -7723592293110705685
    return ((h ^ (h >> 29)) & 0x7FFFFFFF) % maxw + 1


def _sources(u, gen, k):
    """k distinct ends of random edges: in the giant component but for a negligible chance."""
    picked = u[torch.randint(0, u.numel(), (8 * k + 64,), generator=gen, device=DEV)].cpu().numpy()
    return picked[np.sort(np.unique(picked, return_index=True)[1])][:k].astype(np.int32)


def prepare(case, seed):
    row, u, v, gen = _csr(case, seed)
    n = _vertices(case)
    w = _weights(u, v, case["maxw"], n, seed) if "maxw" in case else None
    host = [t.to(torch.int32).cpu().numpy() for t in (row, v)]
    wh = None if w is None else w.to(torch.int32).cpu().numpy().view(np.uint32)
    ctx = gfr.Context(0, tuning_json=gfr.tuned_json() if case["tuned"] else None)
    s = {"op": case["op"], "ctx": ctx, "g": ctx.graph_load_csr(host[0], host[1], wh)}
    op = case["op"]
    if op in ("bfs", "sssp"):
        s["source"] = int(_sources(u, gen, 1)[0])
        s["pred"] = np.empty(n, np.int32) if case["pred"] and case["host"] else case["pred"]
        s["out"] = np.empty(n, np.int32 if op == "bfs" else np.uint32) if case["host"] else None
    elif op in ("bfs_batch", "sssp_batch"):
        s["sources"] = _sources(u, gen, case["k"])
        size = n * s["sources"].size
        s["out"] = np.empty(size, np.int32 if op == "bfs_batch" else np.uint32) if case["host"] else None
    elif op == "bc":
        s["sources"] = _sources(u, gen, case["k"])
    elif op == "pagerank":
        s["tol"] = case["tol"]
    elif op == "step":
        deg = row[1:] - row[:-1]
        s["deg"] = deg.to(torch.int32)
        # random vertices, as many as the buffers hold the edges of
        some = torch.randint(0, n, (case["edges"],), generator=gen, device=DEV)
        some = some[(deg[some] > 0) & (deg[some] <= case["edges"] // 8)]
        s["frontier"] = some[torch.cumsum(deg[some], 0) <= case["edges"]].to(torch.int32)
        visited = torch.rand(n, generator=gen, device=DEV) < 0.3
        visited[s["frontier"].long()] = True
        s["visited"] = visited.to(torch.uint8)
        s["dist"] = torch.randint(0, 1000, (n,), generator=gen, device=DEV).to(torch.int32)
        s["edges"] = torch.full((3, case["edges"]), -1, dtype=torch.int32, device=DEV)
        s["lists"] = torch.full((3, min(n, case["edges"])), -1, dtype=torch.int32, device=DEV)
        s["offs"] = torch.full((min(n, case["edges"]),), -1, dtype=torch.int64, device=DEV)
    return s


# ------------------------------------------------------------------ calls
def run(s):
    ctx, g, op = s["ctx"], s["g"], s["op"]
    if op == "bfs":
        return ctx.bfs(g, s["source"], out=s["out"], pred=s["pred"])
    if op == "sssp":
        return ctx.sssp(g, s["source"], out=s["out"], pred=s["pred"])
    if op == "bfs_batch":
        return ctx.bfs_batch(g, s["sources"], out=s["out"])
    if op == "sssp_batch":
        return ctx.sssp_batch(g, s["sources"], out=s["out"])
    if op == "bc":
        return ctx.bc(g, s["sources"])
    if op == "cc":
        return ctx.cc(g)
    if op == "pagerank":
        rank, iters, l1 = ctx.pagerank(g, 0.85, s["tol"])
        return {"rank": rank, "iters": iters, "l1": np.float32(l1)}
    # one step of a caller's own traversal: expand, cull, prioritise, size the next output
    edges = ctx.advance(g, s["frontier"])
    nxt = ctx.filter(g, edges[2], exclude=s["visited"])
    near, far = ctx.split(g, nxt, s["dist"], 400)
    offs, total = ctx.scan(s["deg"][near])
    for i, t in enumerate(edges):
        s["edges"][i, :t.numel()] = t
    for i, t in enumerate((nxt, near, far)):
        s["lists"][i, :t.numel()] = t
    s["offs"][:offs.numel()] = offs
    return {"edges": s["edges"], "lists": s["lists"], "offs": s["offs"], "total": total}


def work(case):
    """Graph read once, results written once; one operation per edge and query."""
    n, m, op = _vertices(case), _edges(case), case["op"]
    graph = 4 * (n + 1) + 4 * m
    if op in ("bfs", "sssp"):
        return {"bytes": graph + (4 * m if op == "sssp" else 0) + 4 * n * (2 if case["pred"] else 1), "flops": m}
    if op in ("bfs_batch", "sssp_batch"):
        return {"bytes": graph + (4 * m if op == "sssp_batch" else 0) + 4 * n * case["k"], "flops": m * case["k"]}
    if op == "bc":
        return {"bytes": graph + 4 * n, "flops": 2 * m * case["k"]}
    if op in ("cc", "pagerank"):
        return {"bytes": graph + 4 * n, "flops": m}
    e = case["edges"]
    return {"bytes": 8 * e * n // m + 16 * e + 5 * min(e, n), "flops": e}


# -------------------------------------------------------------- reference
def exact(case, seed):
    if case["op"] == "pagerank":
        return _exact_pagerank(case, seed)
    if case["op"] == "bc":
        return _exact_bc(case, seed)
    return None   # whole numbers: depths, distances, labels, lists


def _exact_pagerank(case, seed):
    row, _, v, _ = _csr(case, seed)
    n = _vertices(case)
    deg = (row[1:] - row[:-1]).double()
    x = torch.full((n,), 1.0 / n, dtype=torch.float64, device=DEV)
    for it in range(1, 1001):
        y = torch.where(deg > 0, x / deg.clamp(min=1), 0.0)
        total = torch.segment_reduce(y[v], "sum", offsets=row, initial=0.0)
        nx = 0.15 / n + 0.85 * (total + x[deg == 0].sum() / n)
        l1 = float((nx - x).abs().sum())
        x = nx
        if l1 < case["tol"]:
            break
    return {"rank": x, "iters": None, "l1": l1}


def _row_sums(u, x, n):
    """Sum of x over the edges of each row (u ascending)."""
    offs = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    offs[1:] = torch.cumsum(torch.bincount(u, minlength=n), 0)
    return torch.segment_reduce(x, "sum", offsets=offs, initial=0.0)


def _exact_bc(case, seed):
    row, u, v, gen = _csr(case, seed)
    n = _vertices(case)
    bc = torch.zeros(n, dtype=torch.float64, device=DEV)
    for src in _sources(u, gen, case["k"]).tolist():
        depth = torch.full((n,), GIANT, dtype=torch.int64, device=DEV)
        depth[src] = 0
        sigma = torch.zeros(n, dtype=torch.float64, device=DEV)
        sigma[src] = 1.0
        last = 0
        for level in range(1, n):
            found = v[depth[u] == level - 1]
            found = found[depth[found] == GIANT]
            if found.numel() == 0:
                break
            depth[found] = last = level
            up = (depth[u] == level) & (depth[v] == level - 1)
            sigma += _row_sums(u[up], sigma[v[up]], n)
        delta = torch.zeros(n, dtype=torch.float64, device=DEV)
        for level in range(last - 1, 0, -1):
            down = (depth[u] == level) & (depth[v] == level + 1)
            w = v[down]
            delta += sigma * _row_sums(u[down], (1.0 + delta[w]) / sigma[w], n)
        bc += delta
    return bc
