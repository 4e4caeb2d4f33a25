"""The launch plans of the kernels that take whole chunks (gla_onepass_plan.h, rules on sizes alone), swept on the CPU: what the kernels,
the workspace and the backward pass that takes the states assume of every plan."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2405_18428_amd", "csrc")
SOURCE = r"""
#include "gla_onepass_plan.h"
#include <algorithm>
#include <vector>
using namespace gla;
namespace {
// calls of 1 to 700 sequences (and a few more) of 1 to 1400 chunks, of every kind; false from `holds` ends the sweep
template <typename F> long long sweep(F holds) {
    long long plans = 0;
    for (int small = 0; small < 2; ++small)
        for (int kind = 0; kind < 4; ++kind)            // plain, two-sided, with the prologue, with the epilogue as well
            for (int bh = 1; bh <= 704; ++bh)
                for (int n = 1; n <= 1400; ++n) {
                    const OnePassCall c{bh <= 700 ? bh : 1LL << (bh - 690), n, small != 0, kind == 1, kind >= 2, kind == 3};
                    const OnePassPlan p = onepass_plan(c);
                    if (p.chunks == 0) continue;
                    ++plans;
                    if (!holds(c, p, (n + p.span - 1) / p.span)) return -(((long long)small * 10 + kind) * 100000000LL + bh * 10000LL + n);
                }
    return plans;
}
long long up(long long x) { return (x + 255) / 256 * 256; }
}
extern "C" {
long long shapes() {
    return sweep([](const OnePassCall &c, OnePassPlan p, long long spans) {
        return (p.chunks == 4 || p.chunks == 8) && p.span >= 1 && p.span <= p.chunks && (spans == 1 || p.span > 1) &&
               c.bh * spans * 128 * p.chunks < (1LL << 32) && !(c.two_sided && p.chunks == 8);
    });
}
long long look_back() {
    return sweep([](const OnePassCall &c, OnePassPlan p, long long spans) {
        const bool one_round = c.bh * spans <= (p.chunks == 8 || c.two_sided ? 256 : 512);
        return spans <= kMaxChainedSpans && (spans == 1 || spans <= (one_round ? onepass_most_spans(c, p.chunks) : onepass_most_spans_in_rounds(c, p.chunks)));
    });
}
// Every span is taken once.  Work-group numbers go to the eight XCDs in turn, and an XCD starts its own in order, `resident` of all at a time (one a compute
// unit; two in fours with one gate).  A span's predecessor has a smaller number, of the same XCD or the one before it, or is the last of the XCD range
// before: such waits only go from one range to the one before, so they end, and they are for calls of a round and a half at most.
long long handed_out() {
    std::vector<int> group(1 << 16);
    return sweep([&](const OnePassCall &c, OnePassPlan p, long long spans) {
        const long long blocks = c.bh * spans, resident = p.chunks == 8 || c.two_sided ? 256 : 512;
        if (spans == 1 || blocks > (1 << 16) || (c.bh % 7 > 1 && c.nchunks % 5 > 1)) return spans == 1 || blocks <= (1 << 16);     // (some of them)
        std::fill(group.begin(), group.begin() + blocks, -1);
        for (int b = 0; b < blocks; ++b) {
            const int s = onepass_block(b, (int)blocks, onepass_in_ranges((int)c.bh, (int)spans, onepass_resident(p.chunks, c.two_sided)));
            if (s < 0 || s >= blocks || group[s] >= 0) return false;
            group[s] = b;
        }
        for (int s = 0; s < blocks; ++s) {
            if (s % spans == 0 || group[s - 1] == group[s] - 1 || group[s - 1] == group[s] - 8) continue;
            if (group[s - 1] % 8 != group[s] % 8 - 1 || blocks > resident * 3 / 2) return false;
        }
        return true;
    });
}
// states, sums of the gates and flags of the plan within the bound of one span a chunk (gla_fwd_workspace_bytes)
long long room() {
    return sweep([](const OnePassCall &c, OnePassPlan p, long long spans) {
        for (int h = 0; h < 2 && spans > 1; ++h) {
            const long long dk = c.small ? (h ? 32 : 20) : 36, dv = c.small ? (h ? 64 : 40) : (h ? 72 : 40);
            auto states = [&](long long n) { return up(4 * c.bh * n * dk * dv) + up(4 * c.bh * n * dk) + up(4 * c.bh * n * dv); };
            if (states(spans) + (long long)onepass_flag_bytes(c.bh, spans, p.chunks) > states(c.nchunks) + up(4 * c.bh * c.nchunks)) return false;
        }
        return true;
    });
}
}
"""


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    where = tmp_path_factory.mktemp("plan")
    (where / "plan.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-shared", "-fPIC", "-I", CSRC, "-o", str(where / "plan.so"), str(where / "plan.cpp")],
                   check=True)
    return ctypes.CDLL(str(where / "plan.so"))


@pytest.mark.parametrize("what", ["shapes", "look_back", "handed_out", "room"])
def test_every_plan(plans, what):
    """Groups, spans and threads as the kernels take them; at most as many spans a sequence as its look-back was measured for; no group
    waits for one that is started after it; room for the flags.  (A negative count: kind, sequences and chunks of the first call that breaks it.)"""
    f = getattr(plans, what)
    f.restype = ctypes.c_longlong
    assert f() > 50000
