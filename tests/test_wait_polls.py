"""What a wavefront that waits for several pieces looks at on each poll, on the CPU: a small program built from the library's own header
replays its waits, alone (nobody passes landings on), for every interval between looks at the signals and every phase.
Pieces that have landed, before a wait or together during it, in whichever order they are listed, are seen within one interval for the last one
and one for each wide look that the others take (at once where every poll is a look); a wait whose limit is over looks at everything;
and in between it looks no more often than it may. And those that wait for the same piece take turns."""
import os
import subprocess

import pytest

from paper_2512_10236_amd import _build

PROGRAM = r"""
#include "ficco_internal.h"
#include <algorithm>
#include <cstdio>
#include <vector>
using namespace ficco;

// polls until n pieces are seen; those with bit i of `first` land before the wait, the others before poll `when`
static int wait(int n, uint64_t first, int when, uint32_t every, uint32_t phase)
{
    const uint64_t whole = n == 64 ? ~uint64_t(0) : (uint64_t(1) << n) - 1;
    uint64_t missing = whole;
    PollPlan poll(every, phase);
    for (int p = 1;; ++p) {
        const uint64_t landed = p >= when ? whole : first;
        const int last = 63 - __builtin_clzll(missing);
        uint64_t seen = 0;
        for (int i = 0; i <= last; ++i)
            if ((missing & landed) >> i & 1 && (uint32_t)__builtin_popcountll(missing >> i) <= poll.signals) seen |= uint64_t(1) << i;
        missing &= ~seen;
        if (!missing) return p;
        if (p > 100000) return -1;
        poll.next((int)(seen >> last & 1), 0, (uint32_t)__builtin_popcountll(missing));
    }
}

static int bad(const char *what, int n, int every, int phase, int got)
{
    printf("%s: %d pieces, every %d, phase %d: %d\n", what, n, every, phase, got);
    return 1;
}

// workgroups first, first + step, ... of a launch: on every poll as many of them look at the signals as on any other, give or take `slack`
static int turns(int first, int step, int grid, int every, int slack)
{
    std::vector<int> look(every);
    for (int b = first; b < grid; b += step) ++look[poll_phase((uint32_t)b, (uint32_t)every) % (uint32_t)every];
    const auto mm = std::minmax_element(look.begin(), look.end());
    return *mm.second - *mm.first <= slack ? 0 : bad("turns", step, every, first, *mm.second);
}

int main()
{
    int waits = 0;
    for (int every = 1; every <= 16; ++every)
        for (int grid : {8, 24, 40, 64, 76, 96, 224, 256, 512}) {
            for (int x = 0; x < kTicketLists; ++x)
                if (turns(x, kTicketLists, grid, every, 1)) return 1;
            if (turns(0, 1, grid, every, 4)) return 1;
        }
    for (int every = 1; every <= 16; ++every)
        for (int phase = 0; phase < 256; ++phase)
            for (int n : {1, 2, 3, 4, 8, 16, 63, 64}) {
                const uint64_t whole = n == 64 ? ~uint64_t(0) : (uint64_t(1) << n) - 1;
                const int intervals = 1 + (n - 1 + (int)kLookWide - 1) / (int)kLookWide;
                int p = wait(n, whole, 1, every, phase);
                if (p < 1 || p > (every == 1 ? 1 : intervals * every)) return bad("landed before", n, every, phase, p);
                for (int when : {2, 3, 17, 100}) {
                    for (uint64_t first : {uint64_t(0), whole >> 1, whole & ~uint64_t(1), whole & uint64_t(0xAAAAAAAAAAAAAAAA)}) {
                        p = wait(n, first, when, every, phase);
                        if (p < 0 || p - when >= (every == 1 ? 2 : intervals * every)) return bad("landed during", n, every, phase, p - when);
                        ++waits;
                    }
                }
                PollPlan late(every, phase);
                late.next(0, 0, n); late.next(0, 1, n);
                if (late.signals < (uint32_t)n || !late.flags) return bad("late", n, every, phase, 0);
                if (n <= (int)kLookFew) continue;
                PollPlan poll(every, phase);
                int looks = 0, wide = 0;
                const int polls = 16 * (int)kLookEvery * every;
                for (int i = 0; i < polls; ++i) {
                    poll.next(0, 0, n);
                    looks += poll.signals > 0;
                    wide += poll.signals > 1;
                    if (poll.signals > 1 && !poll.flags) return bad("flags", n, every, phase, i);
                }
                if (looks != 16 * (int)kLookEvery || wide != 16) return bad("looks", n, every, phase, looks);
            }
    printf("%d waits\n", waits);
    return 0;
}
"""


def test_polls_of_a_wait(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    src, exe = tmp_path / "polls.hip", tmp_path / "polls"
    src.write_text(PROGRAM)
    r = subprocess.run([hipcc, "-O1", "-std=c++17", "--offload-host-only", "-I", _build.CSRC, str(src), "-o", str(exe)],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-2000:]
    r = subprocess.run([str(exe)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout
    assert int(r.stdout.split()[0]) > 100000
