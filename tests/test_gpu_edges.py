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
