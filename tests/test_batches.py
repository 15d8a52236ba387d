"""Launch batches of the speculative level loops, compiled for the host: how much
is queued in vain, and how often the host looks.  No device work."""
from __future__ import annotations

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <initializer_list>

#include "batches.h"
using namespace gfr;

// after the first batch: queued in vain less than `share` percent of what was needed (or eight), few looks, no batch
// above 256
template <class Next> constexpr bool good(Next next, int64_t first, int64_t needed, int64_t share)
{
    int64_t launched = first, looks = 1;
    while (launched < needed) {
        const int32_t b = next(launched);
        if (b < 1 || b > 256) return false;
        launched += b;
        ++looks;
    }
    const int64_t bound = needed * share / 100 > 8 ? needed * share / 100 : 8;
    return (launched == first || launched - needed < bound) && looks <= 20 + needed / 200;
}
constexpr bool all()
{
    for (int64_t needed = 1; needed <= 600; ++needed) {
        for (int64_t first : {1, 2, 3, 6, 8, 9, 17, 40, 200})
            if (!good(next_batch, first, needed, 25)) return false;
        for (int64_t first : {1, 5, 8})
            if (!good(next_batch_unknown, first, needed, 67)) return false;
    }
    return good(next_batch, 8, 30000, 25) && good(next_batch_unknown, 8, 30000, 67);
}
static_assert(all(), "");
// never further from the end than doubling from eight, and never twice as many looks
constexpr bool no_worse_than_doubling()
{
    for (int64_t needed = 1; needed <= 600; ++needed) {
        int64_t a = 8, la = 1, d = 8, ld = 1, b = 8;
        while (a < needed) a += next_batch_unknown(a), ++la;
        while (d < needed) d += b = b < 128 ? 2 * b : 256, ++ld;
        if (a > d || la >= 2 * ld + (ld == 1)) return false;
    }
    return true;
}
static_assert(no_worse_than_doubling(), "");
int main() {}
"""


def test_little_is_queued_in_vain(tmp_path):
    src = tmp_path / "batches.cpp"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-fsyntax-only", "-fconstexpr-ops-limit=100000000",
                           "-fconstexpr-loop-limit=1000000", "-Wall", "-I",
                           os.path.join(ROOT, "paper_1501_05387_amd", "csrc"), str(src)])
