"""Steps along a row whose entries are the last ones that an index can name: the
kernels' clamps, compiled for the host.  No device work."""
from __future__ import annotations

import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1501_05387_amd", "csrc")

PROGRAM = r"""
#include "entries.h"
using namespace gfr;

// a row taken `step` entries at a time: ends, names only its own entries, and all of them
constexpr bool walk(uint32_t begin, uint32_t end, uint32_t step)
{
    uint32_t next = begin, turns = 0;
    for (uint32_t e = begin; e < end; e += step) {
        if (++turns > 1000) return false;
        for (uint32_t k = 0; k < step; ++k) {
            const int32_t at = entry_or_last(e, k, end);
            const uint32_t i = (uint32_t)at;
            if (at < 0 || i < begin || i >= end) return false;
            if (e + k < end && i != next++) return false;
        }
    }
    return next == end;
}
constexpr bool walks(uint32_t end)
{
    for (uint32_t len = 0; len <= 70; ++len)
        for (uint32_t step = 4; step <= 32; step *= 2)
            if (!walk(end - len, end, step)) return false;
    return true;
}
constexpr uint32_t LAST = 2147483646u;   // most entries that a graph may have
static_assert(walks(70) && walks(100) && walks(LAST), "");
static_assert(head_end(LAST - 5, LAST, 64) == LAST && head_end(LAST, LAST, 64) == LAST, "");
static_assert(head_end(LAST - 64, LAST, 64) == LAST && head_end(LAST - 65, LAST, 64) == LAST - 1, "");
static_assert(head_end(3, 3, 64) == 3 && head_end(3, 10, 4) == 7, "");
int main() {}
"""


def test_steps_at_the_last_entries(tmp_path):
    src = tmp_path / "entries.cpp"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-fsyntax-only", "-Wall", "-I", CSRC, str(src)])


def test_no_kernel_steps_along_a_row_in_a_signed_index():
    for f in sorted(os.listdir(CSRC)):
        text = open(os.path.join(CSRC, f)).read()
        # an index that starts at a row's offset and then advances by several entries
        for m in re.finditer(r"\bint32_t (\w+) = (?:a\.)?R\[", text):
            assert not re.search(r"\b%s \+= (?!1\b)\d" % m.group(1), text[m.end():m.end() + 1000]), (f, m.group())
