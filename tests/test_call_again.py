"""A call whose wait between work-groups ran out is made once more; any other
failure is the caller's.  The header is compiled for the host; no device work."""
from __future__ import annotations

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "error.h"
using namespace gfr;
void gfr::fail(gfr_status code, const std::string &msg) { throw Error{code, msg}; }
#define CHECK(x) do { if (!(x)) return __LINE__; } while (0)

int main()
{
    for (int crowded = 0; crowded < 2; ++crowded)
        for (int in_order = 0; in_order < 2; ++in_order)
            for (int fails = 0; fails < 3; ++fails) {
                bool first = in_order;
                int calls = 0, got = 0;
                try {
                    call_again_if(
                        [&]() {
                            if (++calls > fails) return;
                            if (crowded) fail_crowded("bfs");
                            fail(GFR_E_DEVICE, "bfs");
                        },
                        [&](const Error &e) {
                            const bool again = e.crowded && first;
                            first = false;
                            return again;
                        });
                } catch (const Error &e) { got = e.code; }
                const bool again = crowded && in_order;
                CHECK(calls == (fails == 0 ? 1 : again ? 2 : 1));
                CHECK(got == (fails > (again ? 1 : 0) ? GFR_E_DEVICE : 0));
            }
    return 0;
}
"""


def test_once_more_where_the_device_was_crowded(tmp_path):
    src, exe = tmp_path / "again.cpp", tmp_path / "again"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-I",
                           os.path.join(ROOT, "paper_1501_05387_amd", "csrc"), "-o", str(exe), str(src)])
    assert subprocess.run([str(exe)], timeout=60).returncode == 0, "line number of the failed check"
