"""GPU parity at the sizes where the solvers change their path: rows, frontiers
and graphs just below, at and above the lines that their dispatch rules draw,
against the CPU oracle."""
from __future__ import annotations

import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_1501_05387_amd as gfr
    c = gfr.Context(0)
    yield c
    c.close()


def _host(t):
    return t.cpu().numpy()


# row lengths around the lane, wave, work-group and step sizes of the scan; hit at the first, a middle and the last entry
PRED_ROWS = [1, 3, 4, 5, 63, 64, 65, 255, 256, 257, 1023, 1024, 1025, 2047, 2048, 2049, 3072, 3073, 4097]


@pytest.mark.parametrize("where", ["first", "middle", "last"])
def test_predecessor_row_lengths(ctx, where):
    eu, ev, leaf = [], [], len(PRED_ROWS)
    hits = []
    for hub, deg in enumerate(PRED_ROWS):
        leaves = np.arange(leaf, leaf + deg)
        leaf += deg
        eu.append(np.full(deg, hub))
        ev.append(leaves)
        hits.append(leaves[{"first": 0, "middle": deg // 2, "last": deg - 1}[where]])
    src = leaf
    eu.append(np.full(len(hits), src))
    ev.append(np.array(hits))
    row, col = graphgen.from_edges(leaf + 1, np.concatenate(eu), np.concatenate(ev))
    w = graphgen.weights(row, col, 64)
    g = ctx.graph_load_csr(row, col, w)
    _, p = ctx.bfs(g, src, pred=True)
    assert np.array_equal(_host(p), oracle.bfs_pred(row, col, src)[1])
    assert np.array_equal(_host(p)[:len(hits)], np.array(hits))
    _, p = ctx.sssp(g, src, pred=True)
    assert np.array_equal(_host(p), oracle.sssp_pred(row, col, w, src)[1])
    g.free()


def _union(*graphs):
    """Disjoint union of CSR graphs, vertices numbered one graph after another."""
    rows, cols, v0, e0 = [np.zeros(1, np.int64)], [], 0, 0
    for row, col in graphs:
        rows.append(row[1:].astype(np.int64) + e0)
        cols.append(col.astype(np.int64) + v0)
        v0 += row.size - 1
        e0 += col.size
    return np.concatenate(rows).astype(np.int32), np.concatenate(cols).astype(np.int32)


def _renumbered(row, col, perm):
    u = np.repeat(np.arange(row.size - 1), np.diff(row))
    keep = u < col
    return graphgen.from_edges(row.size - 1, perm[u[keep]], perm[col[keep]])


CC_GRAPHS = {
    "one vertex": lambda: (np.zeros(2, np.int32), np.zeros(0, np.int32)),
    "no edges": lambda: (np.zeros(301, np.int32), np.zeros(0, np.int32)),
    "pair": lambda: graphgen.from_edges(2, np.array([0]), np.array([1])),
    # no component holds most of the sample: every list is swept, hubs among them
    "two hubs apart": lambda: _union(graphgen.rmat(11, seed=5), graphgen.rmat(11, seed=6),
                                     (np.zeros(70, np.int32), np.zeros(0, np.int32)), graphgen.grid(40)),
    # chains that the first two neighbours leave long, in ascending, descending and mixed order
    "path up": lambda: graphgen.from_edges(70001, np.arange(70000), np.arange(1, 70001)),
    "path mixed": lambda: graphgen.from_edges(*(lambda p: (50021, p[:-1], p[1:]))(
        np.random.default_rng(3).permutation(50021))),
    "lattice mixed": lambda: _renumbered(*graphgen.grid(200), np.random.default_rng(4).permutation(40000)),
    "many small": lambda: graphgen.from_edges(30011, np.arange(0, 30009, 3), np.arange(2, 30011, 3)),
}


@pytest.mark.parametrize("name", list(CC_GRAPHS))
def test_components_of_skipped_and_swept_lists(ctx, name):
    row, col = CC_GRAPHS[name]()
    g = ctx.graph_load_csr(row, col)
    lab, k = ctx.cc(g)
    want, kw = oracle.cc(row, col)
    assert k == kw and np.array_equal(_host(lab), want)
    g.free()


def _tree(arity, depth):
    n = sum(arity ** d for d in range(depth + 1))
    child = np.arange(1, n)
    return graphgen.from_edges(n, (child - 1) // arity, child)


def _at_the_end(n, row, col):
    """The graph as the last vertices of n."""
    lead = n - (row.size - 1)
    return np.concatenate([np.zeros(lead, np.int32), row]), col + np.int32(lead)


MESHES = {   # name: (graph, source)
    "span -1": (lambda: graphgen.from_edges(8191, np.arange(8190), np.arange(1, 8191)), 4000),
    "span": (lambda: graphgen.from_edges(8192, np.arange(8191), np.arange(1, 8192)), 8191),
    "span +1": (lambda: graphgen.from_edges(8193, np.arange(8192), np.arange(1, 8193)), 0),
    # more levels than one launch of the head runs
    "long path": (lambda: graphgen.from_edges(17003, np.arange(17002), np.arange(1, 17003)), 0),
    # 729 vertices discover 6,561: past the head's width and past its list
    "tree": (lambda: _tree(9, 5), 0),
    "ragged lattice": (lambda: graphgen.grid(217), 1234),
    "source without edges": (lambda: _union((np.zeros(41, np.int32), np.zeros(0, np.int32)), graphgen.grid(30)), 7),
    # owners of 32 vertices each
    "wide": (lambda: _at_the_end(8400001, *graphgen.grid(211)), 8400001 - 5),
}


@pytest.mark.parametrize("name", list(MESHES))
def test_mark_byte_levels(ctx, name):
    make, src = MESHES[name]
    row, col = make()
    g = ctx.graph_load_csr(row, col)
    want = oracle.bfs(row, col, src)
    for _ in range(2):
        assert np.array_equal(_host(ctx.bfs(g, src)), want)
        assert ctx.stat("levels") == want.max() + 1
    out = ctx.bfs(g, src)
    assert np.array_equal(_host(ctx.bfs_noalloc(g, src, out)), want)
    g.free()


def test_mark_byte_levels_in_scratch_too_small_for_the_bitmap(ctx):
    n = 33000001   # two mark arrays fit 64 MiB, the visited bitmap does not
    row, col = _at_the_end(n, *graphgen.grid(150))
    g = ctx.graph_load_csr(row, col)
    src = n - 1
    out = ctx.bfs(g, src)
    want = oracle.bfs(row, col, src)
    assert np.array_equal(_host(out), want)
    out.fill_(7)
    assert np.array_equal(_host(ctx.bfs_noalloc(g, src, out)), want)
    g.free()


def _random_regular(n, deg, seed):
    rng = np.random.default_rng(seed)
    u = np.concatenate([rng.permutation(n) for _ in range(deg // 2)])
    v = np.concatenate([rng.permutation(n) for _ in range(deg // 2)])
    return graphgen.from_edges(n, u, v)


@pytest.mark.parametrize("name", list(MESHES))
def test_mark_byte_levels_of_small_graphs(ctx, name):
    """The one-launch levels themselves, also where one work-group would walk the whole graph."""
    import paper_1501_05387_amd as gfr
    make, src = MESHES[name]
    row, col = make()
    g = ctx.graph_load_csr(row, col)
    want = oracle.bfs(row, col, src)
    ctx.set_option("bfs.frontier", 2)
    try:
        for _ in range(2):
            out = ctx.bfs(g, src)
            assert np.array_equal(_host(out), want)
            assert ctx.stat("levels") == want.max() + 1
            with pytest.raises(gfr.GfrError):   # (one work-group reports them)
                ctx.stat("edges_inspected")
        assert np.array_equal(_host(ctx.bfs_noalloc(g, src, out)), want)
        with pytest.raises(gfr.GfrError):
            ctx.stat("edges_inspected")
    finally:
        ctx.set_option("bfs.frontier", 0)
        g.free()


def _ring(n, side):
    """Every vertex joined to `side` neighbours on either side."""
    v = np.arange(n)
    return graphgen.from_edges(n, np.tile(v, side), np.concatenate([(v + d) % n for d in range(1, side + 1)]))


# rows of more than nine entries on average: work-groups of 2,048 vertices, 4,096 from 4,096 vertices per CU on
LONG_ROWS = {   # name: (graph, source)
    "span -1": (lambda: _random_regular(2047, 16, 1), 2046),
    "span": (lambda: _random_regular(2048, 16, 2), 0),
    "span +1": (lambda: _random_regular(2049, 16, 3), 2048),
    "spans": (lambda: _random_regular(30011, 60, 4), 9),
    "ring": (lambda: _ring(20000, 32), 777),
    "near, 4,096": (lambda: _ring(32767, 6), 32766),
    "near, 8,192": (lambda: _ring(32768, 6), 8191),
    "near, 8,192 +1": (lambda: _ring(40961, 6), 40960),
    "larger spans -1": (lambda: _random_regular(1048575, 10, 5), 17),
    "larger spans": (lambda: _random_regular(1048576, 10, 6), 1048575),
    "larger spans +1": (lambda: _random_regular(1048577, 10, 7), 0),
}


@pytest.mark.parametrize("name", list(LONG_ROWS))
def test_mark_byte_levels_over_long_rows(ctx, name):
    make, src = LONG_ROWS[name]
    row, col = make()
    assert col.size > 9 * (row.size - 1)
    g = ctx.graph_load_csr(row, col)
    want = oracle.bfs(row, col, src)
    ctx.set_option("bfs.frontier", 2)
    try:
        for _ in range(2):
            assert np.array_equal(_host(ctx.bfs(g, src)), want)
            assert ctx.stat("levels") == want.max() + 1
    finally:
        ctx.set_option("bfs.frontier", 0)
    assert np.array_equal(_host(ctx.bfs(g, src)), want)
    g.free()


SSSP_MESHES = {   # name: (graph, source, largest weight, bucket width or 0 for the default)
    "span -1": (lambda: graphgen.from_edges(8191, np.arange(8190), np.arange(1, 8191)), 4000, 64, 0),
    "span": (lambda: graphgen.from_edges(8192, np.arange(8191), np.arange(1, 8192)), 8191, 64, 100),
    "span +1": (lambda: graphgen.from_edges(8193, np.arange(8192), np.arange(1, 8193)), 0, 64, 0),
    # more improved vertices than the list of a span has places for
    "one span full": (lambda: _random_regular(8192, 12, 1), 17, 1000, 1000000),
    "spans full": (lambda: _random_regular(40000, 12, 2), 39999, 1000, 1000000),
    "narrow buckets": (lambda: graphgen.grid(217), 1234, 1000, 40),
    "one weight": (lambda: graphgen.grid(120), 5, 1, 0),
    "source without edges": (lambda: _union((np.zeros(41, np.int32), np.zeros(0, np.int32)), graphgen.grid(30)), 7,
                             64, 0),
    # spans of which not all are resident: no rounds in a launch; owners of 32 vertices
    "no rounds": (lambda: _at_the_end(7000001, *graphgen.grid(211)), 7000001 - 5, 1000, 0),
    "wide": (lambda: _at_the_end(8400001, *graphgen.grid(211)), 8400001 - 5, 1000, 0),
}


@pytest.mark.parametrize("name", list(SSSP_MESHES))
def test_mark_byte_iterations(ctx, name):
    make, src, maxw, delta = SSSP_MESHES[name]
    row, col = make()
    w = graphgen.weights(row, col, maxw)
    if name == "narrow buckets":
        w = np.where(w % 5 == 0, np.uint32(0), w).astype(np.uint32)   # (symmetric: the weight depends on the pair)
    g = ctx.graph_load_csr(row, col, w)
    ctx.set_option("sssp.delta", delta)
    ctx.set_option("sssp.frontier", 2 if "full" in name else 0)
    try:
        want = oracle.sssp(row, col, w, src)
        for _ in range(2):
            assert np.array_equal(_host(ctx.sssp(g, src)).view(np.uint32), want)
    finally:
        ctx.set_option("sssp.delta", 0)
        ctx.set_option("sssp.frontier", 0)
        g.free()


def _shuffled(row, col, seed):
    return _renumbered(row, col, np.random.default_rng(seed).permutation(row.size - 1))


# graphs whose edges leave the spans: 2,048 vertices to a work-group, 4,096 from 4,096 vertices per CU on
SSSP_FAR = {   # name: (graph, source, largest weight, bucket width or 0 for the default)
    "span -1": (lambda: _shuffled(*graphgen.from_edges(10239, np.arange(10238), np.arange(1, 10239)), 1), 5, 64, 0),
    "span": (lambda: _shuffled(*graphgen.from_edges(10240, np.arange(10239), np.arange(1, 10240)), 2), 10239, 64, 0),
    "span +1": (lambda: _shuffled(*graphgen.from_edges(10241, np.arange(10240), np.arange(1, 10241)), 3), 0, 64, 100),
    "lattice": (lambda: _shuffled(*graphgen.grid(217), 4), 1234, 1000, 0),
    "narrow buckets": (lambda: _shuffled(*graphgen.grid(120), 5), 77, 1000, 40),
    "wide buckets": (lambda: _random_regular(100003, 6, 6), 9, 1000, 16000),
    "long rows": (lambda: _random_regular(30011, 40, 7), 9, 64, 0),
    "larger spans -1": (lambda: _random_regular(1048575, 4, 8), 17, 64, 0),
    "larger spans": (lambda: _random_regular(1048576, 4, 9), 1048575, 64, 200),
    "larger spans +1": (lambda: _random_regular(1048577, 4, 10), 0, 1000, 0),
}


@pytest.mark.parametrize("name", list(SSSP_FAR))
def test_mark_byte_iterations_across_spans(ctx, name):
    make, src, maxw, delta = SSSP_FAR[name]
    row, col = make()
    w = graphgen.weights(row, col, maxw)
    g = ctx.graph_load_csr(row, col, w)
    ctx.set_option("sssp.delta", delta)
    ctx.set_option("sssp.frontier", 2)
    try:
        want = oracle.sssp(row, col, w, src)
        for _ in range(2):
            assert np.array_equal(_host(ctx.sssp(g, src)).view(np.uint32), want)
    finally:
        ctx.set_option("sssp.delta", 0)
        ctx.set_option("sssp.frontier", 0)
        g.free()


def _rows(degrees, seed):
    """Symmetric simple graph whose first vertices have the given numbers of neighbours (leaves of their own)."""
    eu, ev, leaf = [], [], len(degrees)
    for v, d in enumerate(degrees):
        eu.append(np.full(d, v))
        ev.append(np.arange(leaf, leaf + d))
        leaf += d
    # and some edges among the leaves, so that the sums differ
    rng = np.random.default_rng(seed)
    eu.append(rng.integers(len(degrees), leaf, leaf // 3))
    ev.append(rng.integers(len(degrees), leaf, leaf // 3))
    u, v = np.concatenate(eu), np.concatenate(ev)
    return graphgen.from_edges(leaf, u[u != v], v[u != v])


GATHER_ROWS = {   # list lengths around a lane's four edges, a wave's 256, a chunk's 1024 and the fix-up's eight chunks
    "short": [1, 2, 3, 4, 5, 3, 1, 8, 7, 9, 1, 1, 1, 1],
    "wave": [3, 255, 1, 256, 257, 511, 512, 513, 1, 2],
    "chunk": [1023, 1, 1024, 1025, 2047, 2048, 2049, 5],
    "hubs": [8191, 8192, 8193, 20001, 9 * 1024 + 1, 3],
    "one edge": [1],
    "one chunk": [512],
}


@pytest.mark.parametrize("name", list(GATHER_ROWS))
def test_gathered_sums_of_list_lengths(ctx, name):
    row, col = _rows(GATHER_ROWS[name], 5)
    g = ctx.graph_load_csr(row, col)
    x, it, _ = ctx.pagerank(g, 0.85, 0.0, 6)
    want, _, _ = oracle.pagerank(row, col, 0.85, 0.0, 6)
    assert it == 6 and np.abs(_host(x).astype(np.float64) - want).sum() <= 1e-6
    src = np.array([0, row.size - 2], np.int32)
    b, bo = _host(ctx.bc(g, src)).astype(np.float64), oracle.bc(row, col, src)
    nz = bo != 0
    assert np.all(b[~nz] == 0) and (not nz.any() or np.max(np.abs(b[nz] - bo[nz]) / bo[nz]) <= 1e-5)
    seeds = np.array([0, row.size // 2], np.int32) if row.size > 4 else np.array([0], np.int32)
    hops = _host(ctx.two_hop(g, seeds)).astype(np.uint64)
    assert np.array_equal(hops, oracle.two_hop(row, col, seeds))
    g.free()


def _hubs_and_rest():
    """More than 2^21 entries: list lengths around the 256-edge chunk and the fix-up's 16 chunks, a hub of
    thousands of chunks, isolated vertices, and a ragged number of entries."""
    hubs = _rows([255, 256, 257, 1, 1, 511, 513, 4095, 4096, 4097, 4352, 8191, 40001, 1050007], 9)
    return _union((np.zeros(34, np.int32), np.zeros(0, np.int32)), graphgen.rmat(12), hubs,
                  (np.zeros(78, np.int32), np.zeros(0, np.int32)))


RANKED = {"rmat17": lambda: graphgen.rmat(17), "hubs": _hubs_and_rest}


@pytest.mark.parametrize("name", list(RANKED))
def test_ranked_columns(ctx, name):
    """PageRank over columns renumbered by degree (max_iter >= 4) and over the CSR (below)."""
    row, col = RANKED[name]()
    assert col.size > 1 << 21 and (col.size % 256 or name != "hubs")
    g = ctx.graph_load_csr(row, col)
    held = ctx.graph_info(g)[2]
    for iters in (3, 4, 7):
        x, it, l1 = ctx.pagerank(g, 0.85, 0.0, iters)
        assert (ctx.graph_info(g)[2] > held) == (iters > 3)
        want, _, wl1 = oracle.pagerank(row, col, 0.85, 0.0, iters)
        x = _host(x).astype(np.float64)
        assert it == iters and np.abs(x - want).sum() <= 1e-6
        assert np.all(np.abs(x - want) <= 1e-5 * want) and abs(l1 - wl1) <= 1e-6
    out = np.empty(row.size - 1, np.float32)
    _, it, l1 = ctx.pagerank(g, 0.85, 1e-6, 1000, out=out)
    again, it2, l2 = ctx.pagerank(g, 0.85, 1e-6, 1000)
    assert it == it2 and l1 == l2 < 1e-6 and np.array_equal(out, _host(again))
    g.free()


# scale, edge factor, (iterations, tolerance) of the calls, which of them hold the ranked columns afterwards
RANKED_CALLS = {
    "small": (17, 16, [(1000, 1e-6), (3, 0.0), (4, 0.0)], [False, False, True]),
    "first call": (18, 32, [(8, 0.0)], [True]),
    "few iterations": (18, 32, [(7, 0.0), (4, 0.0)], [False, True]),
    "loose": (18, 32, [(1000, 1e-2), (1000, 0.5)], [False, True]),
}


@pytest.mark.parametrize("name", list(RANKED_CALLS))
def test_the_call_that_makes_ranked_columns(ctx, name):
    """Only where the call itself is faster with them, or when the graph is ranked again."""
    scale, factor, calls, want = RANKED_CALLS[name]
    row, col = graphgen.rmat(scale, factor)
    assert (1 << 21 if name == "small" else 10 << 20) < col.size < (10 << 20 if name == "small" else 1 << 25)
    g = ctx.graph_load_csr(row, col)
    held = ctx.graph_info(g)[2]
    got = []
    for iters, tol in calls:
        _, it, _ = ctx.pagerank(g, 0.85, tol, iters)
        got.append(ctx.graph_info(g)[2] > held)
        assert it <= iters
    assert got == want
    g.free()


def _without_rows(row, col, drop):
    """The graph without the rows of the vertices in `drop`; entries that name them stay."""
    deg = np.diff(row)
    keep = ~np.repeat(drop, deg)
    return np.concatenate([[0], np.cumsum(np.where(drop, 0, deg))]).astype(np.int32), col[keep]


def _pagerank(row, col, damping, iters):
    """Power iteration in float64; a vertex without edges gives its rank to all, and nothing to those that name it."""
    n, deg = row.size - 1, np.diff(row)
    rows, x = np.repeat(np.arange(n), deg), np.full(n, 1.0 / n)
    for _ in range(iters):
        y = np.where(deg > 0, x / np.maximum(deg, 1), 0.0)
        total = np.bincount(rows, weights=y[col], minlength=n)
        x = (1 - damping) / n + damping * (total + x[deg == 0].sum() / n)
    return x


@pytest.mark.parametrize("share", [0.1, 0.97])   # (0.97: every value of the table fits LDS)
def test_pagerank_of_targets_without_edges(ctx, share):
    """An asymmetric graph is accepted when no validation is asked for: its columns name vertices without a row."""
    row, col = graphgen.rmat(18, 32)
    deg = np.diff(row)
    drop = np.random.default_rng(8).random(row.size - 1) < share
    drop[np.argsort(deg)[-3000:]] = False   # the hubs keep the entries over the ranked columns' line
    row, col = _without_rows(row, col, drop)
    assert np.any(np.diff(row)[col] == 0) and col.size > 1 << 21
    g = ctx.graph_load_csr(row, col)
    for iters in (3, 9, 9):   # over the CSR, then over the ranked columns
        x = _host(ctx.pagerank(g, 0.85, 0.0, iters)[0]).astype(np.float64)
        want = _pagerank(row, col, 0.85, iters)
        assert np.abs(x - want).sum() <= 1e-6 and np.all(np.abs(x - want) <= 1e-5 * want)
    g.free()


SMALL = {   # name: (graph, source): around the rules of the one-work-group traversal, both lane counts
    "one vertex": (lambda: (np.zeros(2, np.int32), np.zeros(0, np.int32)), 0),
    "no edges at the source": (lambda: _union((np.zeros(6, np.int32), np.zeros(0, np.int32)), graphgen.rmat(9)), 2),
    "row at the hub's line": (lambda: _rows([511, 512, 513, 1025, 3], 1), 0),
    "hub": (lambda: _rows([60000, 700], 2), 60001),
    "rmat": (lambda: graphgen.rmat(12), 5),
    "most vertices": (lambda: graphgen.from_edges(32768, np.arange(32767), np.arange(1, 32768)), 32767),
    "past the list": (lambda: graphgen.from_edges(32769, np.arange(32768), np.arange(1, 32769)), 3),
    "row of 16": (lambda: _rows([16, 16, 1, 15], 3), 0),
    "row of 17": (lambda: _rows([17, 16, 1, 15], 3), 0),
    "lattice": (lambda: graphgen.grid(181), 77),
}


@pytest.mark.parametrize("name", list(SMALL))
def test_small_graph_bfs(ctx, name):
    make, src = SMALL[name]
    row, col = make()
    g = ctx.graph_load_csr(row, col)
    want = oracle.bfs(row, col, src)
    for direction in (0, 1, 2):
        ctx.set_option("bfs.direction", direction)
        try:
            d = ctx.bfs(g, src)
        finally:
            ctx.set_option("bfs.direction", 0)
        assert np.array_equal(_host(d), want)
        if direction < 2 and row[src + 1] > row[src]:
            assert ctx.stat("levels") == want.max() + 1
    assert np.array_equal(_host(ctx.bfs_noalloc(g, src, d)), want)
    g.free()


@pytest.mark.parametrize("n, side, one_group", [(32768, 4, True), (32769, 4, False), (19661, 6, True),
                                                (19662, 6, False), (16384, 8, True), (16385, 8, False)])
def test_small_graph_bfs_line_by_row_length(ctx, n, side, one_group):
    """One work-group as long as the entries it walks alone are few; the one-launch levels report no edges."""
    import paper_1501_05387_amd as gfr
    row, col = _ring(n, side)
    g = ctx.graph_load_csr(row, col)
    for src in (0, n - 1):
        assert np.array_equal(_host(ctx.bfs(g, src)), oracle.bfs(row, col, src))
        if one_group:
            assert ctx.stat("edges_inspected") == col.size and ctx.stat("launches") == 1
        else:
            with pytest.raises(gfr.GfrError):
                ctx.stat("edges_inspected")
    g.free()


# what the queue levels and iterations report, and so every path that is taken in their place
BFS_STATS = ["levels", "push_levels", "pull_levels", "edges_inspected", "push_entries", "push_edges", "push_new",
             "pull_unvisited", "pull_inspected", "pull_new", "launches", "solves", "kernel_ms"]
SSSP_STATS = ["iterations", "relaxations", "edges_inspected", "splits", "near_entries", "improvements",
              "far_entries", "pull_iterations", "delta", "launches", "solves", "kernel_ms"]


def test_statistics_of_the_paths_without_a_queue(ctx):
    row, col = _union((np.zeros(6, np.int32), np.zeros(0, np.int32)), graphgen.rmat(11))
    g = ctx.graph_load_csr(row, col)
    src = int(np.argmax(np.diff(row)))
    got = []
    for frontier in (1, 0):   # queue levels; one work-group
        ctx.set_option("bfs.frontier", frontier)
        ctx.set_option("bfs.direction", 1)
        try:
            ctx.bfs(g, src)
            got.append({k: ctx.stat(k) for k in BFS_STATS})
            ctx.bfs(g, 2)     # no edges at the source
            got[-1]["levels without edges"] = ctx.stat("levels")
        finally:
            ctx.set_option("bfs.frontier", 0)
            ctx.set_option("bfs.direction", 0)
    for s in got:
        del s["kernel_ms"], s["launches"]
    assert got[0] == got[1]
    g.free()
    row, col = graphgen.grid(60)
    g = ctx.graph_load_csr(row, col, graphgen.weights(row, col, 64))
    for frontier in (1, 2):
        ctx.set_option("sssp.frontier", frontier)
        try:
            ctx.sssp(g, 7)
            assert all(ctx.stat(k) >= 0 for k in SSSP_STATS) and ctx.stat("pull_iterations") == 0
        finally:
            ctx.set_option("sssp.frontier", 0)
    g.free()


@pytest.mark.parametrize("k", [2, 24, 31, 32, 33, 64, 65, 97])
@pytest.mark.parametrize("name", ["rmat", "hub rows", "lattice", "no edges at a source"])
def test_batches_part_filled(ctx, name, k):
    """Batches of every fill, duplicated sources among them, on graphs of one chunk and of many."""
    row, col = {"rmat": lambda: graphgen.rmat(13), "hub rows": lambda: _rows([255, 256, 257, 1024, 1025, 3, 9000], 4),
                "lattice": lambda: graphgen.grid(70),
                "no edges at a source": lambda: _union((np.zeros(4, np.int32), np.zeros(0, np.int32)),
                                                       graphgen.rmat(9))}[name]()
    n = row.size - 1
    w = graphgen.weights(row, col, 64)
    g = ctx.graph_load_csr(row, col, w)
    src = np.random.default_rng(k).integers(0, n, k).astype(np.int32)
    src[-1] = src[0]
    if name == "no edges at a source":
        src[k // 2] = 1
    ctx.set_option("batch.min_sssp", 2)
    ctx.set_option("batch.min_bfs", 2)
    try:
        for delta in (0, 70):
            ctx.set_option("batch.delta", delta)
            d = _host(ctx.sssp_batch(g, src)).view(np.uint32).reshape(k, n)
            for i in set([0, 1, k // 2, k - 2, k - 1]):
                assert np.array_equal(d[i], oracle.sssp(row, col, w, int(src[i])))
        b = _host(ctx.bfs_batch(g, src)).reshape(k, n)
        for i in set([0, 1, k // 2, k - 1]):
            assert np.array_equal(b[i], oracle.bfs(row, col, int(src[i])))
    finally:
        ctx.set_option("batch.delta", 0)
        ctx.set_option("batch.min_sssp", 24)
        ctx.set_option("batch.min_bfs", 8)
        g.free()


@pytest.mark.parametrize("count", [1, 2047, 2048, 2049, 2048 * 1024, 2048 * 1024 + 1])
def test_operator_lists_at_tile_edges(ctx, count):
    """Lists of one tile to one past what every work-group sums itself; a bad last id or a list that
    does not fit leaves the outputs as they were."""
    import ctypes
    import torch
    import paper_1501_05387_amd as gfr
    n = max(count, 8)                                     # filter scans the vertices, the others the list
    row = np.zeros(n + 1, np.int32)
    row[-1] = 2                                           # the last vertex has two edges
    col = np.array([0, n - 2], np.int32)
    g = ctx.graph_load_csr(row, col)
    X = np.random.default_rng(count).permutation(n).astype(np.int32) if count == n else np.array([n - 1], np.int32)
    src, edge, dst = (np.full(2, n - 1, np.int32), np.arange(2, dtype=np.int32), col)
    for got, want in zip(ctx.advance(g, torch.from_numpy(X).cuda()), (src, edge, dst)):
        assert np.array_equal(_host(got), want)
    assert np.array_equal(_host(ctx.filter(g, X)), np.sort(X))
    dist = (np.arange(n) % 5).astype(np.uint32)
    near, far = ctx.split(g, X, dist, 2)
    assert np.array_equal(_host(near), X[dist[X] < 2]) and np.array_equal(_host(far), X[dist[X] >= 2])
    outs = [torch.full((count + 2,), -7, dtype=torch.int32, device="cuda") for _ in range(3)]
    a, b, c = (o.data_ptr() for o in outs)
    k, k2 = ctypes.c_int64(), ctypes.c_int64()
    L = gfr.lib()

    def calls(items, cap):
        i = items.ctypes.data
        return (L.gfr_advance(ctx.ptr, g.handle, i, count, a, b, c, min(cap, 1), ctypes.byref(k), None),
                L.gfr_filter(ctx.ptr, g.handle, i, count, None, a, cap, ctypes.byref(k), None),
                L.gfr_split(ctx.ptr, g.handle, i, count, dist.ctypes.data, 9, a, b, cap, ctypes.byref(k),
                            ctypes.byref(k2), None))

    assert calls(X, count - 1) == (gfr.GFR_E_CAPACITY,) * 3
    for bad in (n, -1):
        Y = X.copy()
        Y[-1] = bad
        assert calls(Y, count + 2) == (gfr.GFR_E_INVALID,) * 3
    torch.cuda.synchronize()
    assert all(bool((o == -7).all()) for o in outs)
    g.free()


def test_results_are_complete_on_return(ctx):
    """Two contexts in two threads, short and long solves in turn, each result read at once on another stream."""
    import threading
    import torch
    import paper_1501_05387_amd as gfr
    row, col = graphgen.rmat(10)
    lrow, lcol = graphgen.grid(400)
    w = graphgen.weights(lrow, lcol, 64)
    want = [oracle.bfs(row, col, s) for s in range(8)]
    long = [oracle.sssp(lrow, lcol, w, s) for s in (0, 1)]
    X = np.arange(0, row.size - 1, 3, dtype=np.int32)
    bad = []

    def work():
        c, st = gfr.Context(0), torch.cuda.Stream()
        g, lg = c.graph_load_csr(row, col), c.graph_load_csr(lrow, lcol, w)
        with torch.cuda.stream(st):
            for i in range(40):
                got = c.bfs(g, i % 8).clone()
                kept = c.filter(g, X).clone()
                d = c.sssp(lg, i % 2).clone() if i % 10 == 0 else None
                if not (np.array_equal(_host(got), want[i % 8]) and np.array_equal(_host(kept), X)):
                    bad.append(i)
                if d is not None and not np.array_equal(_host(d).view(np.uint32), long[i % 2]):
                    bad.append(-i)
        c.close()

    ts = [threading.Thread(target=work) for _ in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad


def _hubs(rows, tail=0):
    """Vertex 0 beside hubs 1..len(rows), hub i beside its own rows[i] - 1 leaves, `tail` vertices after
    them in a chain that starts at the last leaf."""
    k, first = len(rows), len(rows) + 1
    eu, ev = [np.zeros(k, np.int64)], [np.arange(1, k + 1)]
    for i, r in enumerate(rows):
        eu.append(np.full(r - 1, i + 1))
        ev.append(np.arange(first, first + r - 1))
        first += r - 1
    eu.append(np.arange(first - 1, first - 1 + tail))
    ev.append(np.arange(first, first + tail))
    return graphgen.from_edges(first + tail, np.concatenate(eu).astype(np.int32), np.concatenate(ev).astype(np.int32))


# one word a thread up to 2^22 vertices on 256 CUs, several past it; rows at the chunk size, many chunks a thread
QUEUES = {
    "chunk rows": lambda: _hubs([1024, 1, 1023, 1, 1025, 2, 2048, 1024] * 9, 40),
    "neighbouring hubs": lambda: _hubs([9000] * 64, 40),
    "word ends": lambda: _hubs([2] * 2047, 33),
    "one word a thread": lambda: _hubs([1 << 21, (1 << 21) - 4], 3),
    "two words a thread": lambda: _hubs([1 << 21, (1 << 21) + 60], 3),
}


@pytest.mark.parametrize("name", list(QUEUES))
def test_queues_at_chunk_and_word_edges(ctx, name):
    row, col = QUEUES[name]()
    g = ctx.graph_load_csr(row, col)
    n = row.size - 1
    ctx.set_option("bfs.frontier", 1)
    ctx.set_option("bfs.direction", 1)
    try:
        for src in (0, 1, n - 1):
            assert np.array_equal(_host(ctx.bfs(g, src)), oracle.bfs(row, col, src))
    finally:
        ctx.set_option("bfs.frontier", 0)
        ctx.set_option("bfs.direction", 0)
        g.free()


@pytest.mark.parametrize("array", [False, True], ids=["lists", "likely neighbours"])
@pytest.mark.parametrize("last", [True, False], ids=["hit at the end", "hit first"])
def test_pull_list_lengths(ctx, last, array):
    """Lists around the lane's and the quarter wave's steps, whole waves of them and mixed, found at level 2
    through their one frontier neighbour."""
    kinds = [1, 2, 3, 4, 5, 7, 8, 9, 10, 39, 40, 41, 72, 73, 300]
    lens = np.concatenate([np.repeat(k, 64) for k in kinds] + [np.tile(kinds, 9)])
    leaves, w = int((lens - 1).sum()), lens.size
    own = np.repeat(np.arange(w), lens - 1)
    if last:      # leaves, the vertices, their common neighbour x, the source
        w0, x, src, l0 = leaves, leaves + w, leaves + w + 1, 0
    else:         # the source, x, the vertices, leaves
        w0, x, src, l0 = 2, 1, 0, 2 + w
    eu = np.concatenate([w0 + own, w0 + np.arange(w), [x]])
    ev = np.concatenate([l0 + np.arange(leaves), np.full(w, x), [src]])
    row, col = graphgen.from_edges(leaves + w + 2, eu.astype(np.int32), ev.astype(np.int32))
    if array:     # enough entries beside them that the array is made
        row, col = _union((row, col), _hubs([1 << 21, (1 << 21) + 60], 3))
    g = ctx.graph_load_csr(row, col)
    ctx.set_option("bfs.frontier", 1)
    ctx.set_option("bfs.direction", 2)
    try:
        for s in (src, l0, w0 + w - 1):
            assert np.array_equal(_host(ctx.bfs(g, int(s))), oracle.bfs(row, col, int(s)))
    finally:
        ctx.set_option("bfs.frontier", 0)
        ctx.set_option("bfs.direction", 0)
        g.free()


def test_outputs_queued_before_the_end_is_known(ctx):
    """A solve longer than the launches queued at first: the output kernels run again once it has ended."""
    row, col = graphgen.grid(60)          # 119 levels, after a star's two
    w = graphgen.weights(row, col, 64)
    star, scol = graphgen.from_edges(70, np.zeros(69, np.int32), np.arange(1, 70, dtype=np.int32))
    row, col = _union((star, scol), (row, col))
    w = np.concatenate([np.ones(scol.size, np.uint32), w])
    g = ctx.graph_load_csr(row, col, w)
    for first in (0, 100):                # sources in the star, then in the lattice
        src = (np.arange(30, dtype=np.int32) + first)
        for _ in range(2):
            b = _host(ctx.bfs_batch(g, src)).reshape(30, -1)
            d = _host(ctx.sssp_batch(g, src)).view(np.uint32).reshape(30, -1)
            for i in (0, 13, 29):
                assert np.array_equal(b[i], oracle.bfs(row, col, int(src[i])))
                assert np.array_equal(d[i], oracle.sssp(row, col, w, int(src[i])))
    g.free()


@pytest.mark.parametrize("degree", [8, 10, 34])
def test_regular_graph_bfs_around_the_mark_byte_line(ctx, degree):
    n, rng = 40009, np.random.default_rng(degree)
    rings = [rng.permutation(n) for _ in range(degree // 2)]
    row, col = graphgen.from_edges(n, np.concatenate(rings).astype(np.int32),
                                   np.concatenate([np.roll(p, 1) for p in rings]).astype(np.int32))
    g = ctx.graph_load_csr(row, col)
    for src in (0, n - 1):
        want = oracle.bfs(row, col, src)
        d = ctx.bfs(g, src)
        assert np.array_equal(_host(d), want)
        assert np.array_equal(_host(ctx.bfs_noalloc(g, src, d)), want)
    g.free()


def _sparse(n, m, seed):
    rng = np.random.default_rng(seed)
    return graphgen.from_edges(n, rng.integers(0, n, m), rng.integers(0, n, m))


@pytest.mark.parametrize("n", [8192, 8193, 300007, 4194304, 4194369])
def test_compactions_placed_by_their_start(ctx, n):
    """Beside another context's call the work-groups take their places as they start; the results stay."""
    import threading
    import paper_1501_05387_amd as gfr
    row, col = _sparse(n, 2 * n, n)   # one work-group, two, 37, 512 and two words a thread
    w = graphgen.weights(row, col, 64)
    srcs = graphgen.sample_sources(row, col, 3)
    prow, pcol = graphgen.from_edges(20000, np.arange(19999), np.arange(1, 20000))
    stop, ran = threading.Event(), []

    def beside(c):   # calls of 20,000 levels, one after the other
        g = c.graph_load_csr(prow, pcol)
        c.set_option("bfs.frontier", 1)
        while not stop.is_set():
            ran.append(int(c.bfs(g, 0).max()))

    g = ctx.graph_load_csr(row, col, w)
    ctx.set_option("bfs.frontier", 1)
    ctx.set_option("sssp.frontier", 1)
    try:
        with gfr.Context(0) as other:
            got = []
            for crowd in (False, True):
                t = threading.Thread(target=beside, args=(other,)) if crowd else None
                if t:
                    t.start()
                    while not ran:
                        stop.wait(0.01)
                out = [_host(ctx.bfs(g, int(srcs[0]))), _host(ctx.sssp(g, int(srcs[1]))).view(np.uint32),
                       _host(ctx.bfs_batch(g, srcs)), _host(ctx.sssp_batch(g, srcs)), _host(ctx.bc(g, srcs[:2])),
                       _host(ctx.two_hop(g, srcs)), _host(ctx.pagerank_filtered(g, 0.85, 1e-4 / n, 30)[0])]
                if t:
                    stop.set()
                    t.join()
                got.append(out)
            assert set(ran) == {19999}
    finally:
        stop.set()
        ctx.set_option("bfs.frontier", 0)
        ctx.set_option("sssp.frontier", 0)
        g.free()
    assert np.array_equal(got[0][0], oracle.bfs(row, col, int(srcs[0])))
    assert np.array_equal(got[0][1], oracle.sssp(row, col, w, int(srcs[1])))
    for a, b in zip(*got):
        assert np.array_equal(a, b)


def test_compactions_of_contexts_side_by_side(ctx):
    """Grids that each fill the chip wait inside themselves only: no context's look-back runs out."""
    import threading
    import torch
    import paper_1501_05387_amd as gfr
    row, col = _sparse(4194304, 4194304, 11)
    src = int(graphgen.sample_sources(row, col, 1)[0])
    want = torch.from_numpy(oracle.bfs(row, col, src)).cuda()
    wrong = []

    def calls(c, k):
        g = c.graph_load_csr(row, col)
        c.set_option("bfs.frontier", 1)
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for i in range(30):
                    out = c.bfs(g, src) if i % 3 else c.bfs_batch(g, [src])
                    if not torch.equal(out.view(-1), want):
                        wrong.append((k, i))
        except Exception as e:   # a look-back that ran out
            wrong.append((k, str(e)))
        finally:
            c.set_option("bfs.frontier", 0)
            g.free()

    with gfr.Context(0) as second, gfr.Context(0) as third:
        threads = [threading.Thread(target=calls, args=(c, k)) for k, c in enumerate((ctx, second, third))]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
    assert not wrong
