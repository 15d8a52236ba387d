"""The lane arithmetic of the segmented gather, restated: which entry of a queue,
and which place in the columns, each of a chunk's edge slots reads.  Slots past
the last edge must read that edge again, whatever the order of the queue's rows."""
from __future__ import annotations

import os
import re

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CH, EPL = 1024, 4


def _delta_index():
    """The entry whose delta a slot adds, as the kernel's source has it, as a function of (slot is an edge, entry)."""
    text = open(os.path.join(ROOT, "paper_1501_05387_amd", "csrc", "gather.h")).read()
    expr = re.search(r"u\[j\] = C\[\(int32_t\)e \+ s_delta\[(.*)\]\];", text).group(1)
    if expr == "ent[j]":
        return lambda edge, ent: ent
    assert expr == "e0 + k + j < e1 ? ent[j] : 0", expr
    return lambda edge, ent: np.where(edge, ent, 0)


@pytest.mark.parametrize("order", ["ascending", "descending", "mixed"])
@pytest.mark.parametrize("total", [1, 3, 255, 1023, 1024, 1025, 2500])
def test_slots_past_the_last_edge_read_it_again(order, total):
    rng = np.random.default_rng(total)
    deg = np.minimum(rng.integers(1, 60, total), 700)
    deg = deg[:np.searchsorted(np.cumsum(deg), total) + 1]
    deg[-1] -= deg.sum() - total
    starts = np.concatenate([[0], np.cumsum(deg)[:-1]])   # rows as they lie in the columns
    pick = {"ascending": np.arange(deg.size), "descending": np.arange(deg.size)[::-1],
            "mixed": rng.permutation(deg.size)}[order]
    row, d = starts[pick], deg[pick]
    off = np.concatenate([[0], np.cumsum(d)[:-1]])
    place = np.repeat(row - off, d) + np.arange(total)    # place in the columns of every edge of the queue
    index = _delta_index()
    for e0 in range(0, total, CH):
        e1 = min(e0 + CH, total)
        first = np.searchsorted(off, e0, side="right") - 1
        slot = e0 + np.arange(CH)
        started = (off >= e0) & (off < e1)
        # entries started up to each slot, less the first one when it starts the chunk
        ent = np.searchsorted(off[started], slot, side="right") - (off[first] == e0)
        edge = slot < e1
        e = np.minimum(slot, e1 - 1)
        reads = e + (row - off)[first + index(edge, ent)]
        assert np.array_equal(reads, place[e])
