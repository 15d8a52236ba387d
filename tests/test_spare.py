"""A structure that only makes calls faster: what the calls find after a failure
while it was being made, and a call that runs out of memory while one is held.
The header is compiled for the host; no device work."""
from __future__ import annotations

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <stdexcept>
#include "spare.h"
using namespace gfr;
void gfr::fail(gfr_status code, const std::string &msg) { throw Error{code, msg}; }

struct Columns {
    Spare have;
    bool allocated = false, filled = false;
    int made = 0;
    // fails after the allocation with `code` (0: not at all)
    bool get(int code)
    {
        const bool there = have.get(
            [&]() {
                ++made;
                allocated = true;
                if (code == 1) throw std::runtime_error("build");
                if (code) fail((gfr_status)code, "build");
                filled = true;
            },
            [&]() { allocated = filled = false; });
        if (there && !(allocated && filled)) throw std::logic_error("a half-made structure was handed out");
        return there;
    }
};
#define CHECK(x) do { if (!(x)) return __LINE__; } while (0)

int main()
{
    {   // no room: the call goes on without it, and so do later ones
        Columns c;
        CHECK(!c.get(GFR_E_OOM) && !c.allocated);
        CHECK(!c.get(0) && c.made == 1);
    }
    for (int code : {(int)GFR_E_DEVICE, 1}) {   // another failure is the caller's; the next call makes it
        Columns c;
        bool thrown = false;
        try { c.get(code); } catch (const Error &) { thrown = true; } catch (const std::runtime_error &) { thrown = true; }
        CHECK(thrown && !c.allocated);
        CHECK(c.get(0) && c.made == 2);
        CHECK(c.get(GFR_E_DEVICE) && c.made == 2);
    }
    {   // a call without room runs again once something was given back
        int calls = 0, freed = 0;
        with_room([&]() { if (++calls == 1) fail(GFR_E_OOM, ""); }, [&]() { ++freed; return true; });
        CHECK(calls == 2 && freed == 1);
    }
    for (int code : {(int)GFR_E_OOM, (int)GFR_E_INVALID}) {   // nothing to give back, or not for want of room
        int calls = 0, freed = 0, got = 0;
        try {
            with_room([&]() { ++calls; fail((gfr_status)code, ""); }, [&]() { ++freed; return false; });
        } catch (const Error &e) { got = e.code; }
        CHECK(calls == 1 && got == code && freed == (code == GFR_E_OOM));
    }
    {   // it fails for good the second time
        int calls = 0, got = 0;
        try {
            with_room([&]() { ++calls; fail(GFR_E_OOM, ""); }, [&]() { return true; });
        } catch (const Error &e) { got = e.code; }
        CHECK(calls == 2 && got == GFR_E_OOM);
    }
    return 0;
}
"""


def test_a_half_made_structure_is_given_back(tmp_path):
    src, exe = tmp_path / "spare.cpp", tmp_path / "spare"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-I",
                           os.path.join(ROOT, "paper_1501_05387_amd", "csrc"), "-o", str(exe), str(src)])
    assert subprocess.run([str(exe)], timeout=60).returncode == 0, "line number of the failed check"
