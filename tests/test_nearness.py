"""Share of a graph's entries between neighbouring ids (it picks the form of the
mark-byte SSSP iterations), compiled for the host.  No device work."""
from __future__ import annotations

import ctypes
import os
import subprocess

import numpy as np
import pytest

import graphgen

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
RUN = 8192


@pytest.fixture(scope="module")
def near(tmp_path_factory):
    d = tmp_path_factory.mktemp("near")
    (d / "near.cpp").write_text('#include "nearness.h"\nextern "C" double near(int32_t n, int64_t m, const int32_t *R, '
                                'const int32_t *C) { return gfr::near_share(n, m, R, C); }\n')
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-Wall", "-I",
                           os.path.join(ROOT, "paper_1501_05387_amd", "csrc"), "-o", str(d / "near.so"),
                           str(d / "near.cpp")])
    f = ctypes.CDLL(str(d / "near.so")).near
    f.restype = ctypes.c_double
    f.argtypes = [ctypes.c_int32, ctypes.c_int64, ctypes.c_void_p, ctypes.c_void_p]
    return lambda row, col: f(row.size - 1, col.size, row.ctypes.data, col.ctypes.data)


def _spread(share, n):
    """Four standard deviations of the samples taken."""
    return 4 * np.sqrt(share * (1 - share) / min(1024, max(256, n // 128))) + 0.01


def _share(row, col):
    u = np.repeat(np.arange(row.size - 1), np.diff(row))
    return np.mean(u // RUN == col // RUN)


@pytest.mark.parametrize("side", [33, 91, 200, 700])
def test_sampled_share_of_lattices_and_shuffled_ones(near, side):
    row, col = graphgen.grid(side)
    n = row.size - 1
    want = 1.0 if n <= RUN else _share(row, col)
    assert abs(near(row, col) - want) < _spread(want, n) and near(row, col) > 0.84
    p = np.random.default_rng(2).permutation(n)
    u = np.repeat(np.arange(n), np.diff(row))
    keep = u < col
    row, col = graphgen.from_edges(n, p[u[keep]], p[col[keep]])
    want = 1.0 if n <= RUN else _share(row, col)
    assert abs(near(row, col) - want) < _spread(want, n)
    assert (near(row, col) < 0.84) == (want < 0.84)


@pytest.mark.parametrize("m", [0, 1, 5, 4095, 4096, 4097, 70001])
def test_few_entries_and_leading_empty_rows(near, m):
    n = 100000
    row = np.zeros(n + 1, np.int32)
    row[n - 10:] = np.linspace(0, m, 11).astype(np.int32)   # the last ten rows hold them all
    far = np.zeros(m, np.int32)
    assert near(row, np.full(m, n - 1, np.int32)) == 1.0
    assert near(row, far) == (1.0 if m == 0 else 0.0)
    if m > 1000:
        assert abs(near(row, np.where(np.arange(m) % 2, n - 1, 0).astype(np.int32)) - 0.5) < _spread(0.5, n)


@pytest.mark.parametrize("side", [128, 512])
def test_rows_that_repeat(near, side):
    """A torus: every row has the same four entries, two of them a row of the torus away."""
    n = side * side
    v = np.arange(n).reshape(side, side)
    u = np.concatenate([v.ravel()] * 2)
    w = np.concatenate([np.roll(v, -1, 0).ravel(), np.roll(v, -1, 1).ravel()])
    row, col = graphgen.from_edges(n, u, w)
    assert np.all(np.diff(row) == 4)
    # renumbered so that a row of the torus is half a run away: two entries of each row leave it every other time
    far = (np.arange(n) * 4096) % n + np.arange(n) * 4096 // n
    if n > 8192:
        row, col = graphgen.from_edges(n, far[u], far[w])
    assert abs(near(row, col) - _share(row, col)) < _spread(_share(row, col), n)
