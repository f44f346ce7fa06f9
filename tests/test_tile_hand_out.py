"""How a short resident launch hands out its tiles, on the CPU: a small program built from the library's own header walks
every workgroup's places over lists that are even, uneven, empty or started by nobody. Every tile is taken exactly once,
by no workgroup more than its share, and no counter is booked; where tiles wait for pieces, nobody takes a tile of another
list behind one of its own. Longer launches book the draws that their lists need."""
import os
import subprocess

import pytest

from paper_2512_10236_amd import _build

PROGRAM = r"""
#include "ficco_internal.h"
#include <cstdio>
#include <vector>
using namespace ficco;

static int bad(const char *what, int64_t rt, int64_t tn, int cl, int grid)
{
    printf("%s: %lld row tiles, %lld column tiles, %d column lists, grid %d\n", what, (long long)rt, (long long)tn, cl, grid);
    return 1;
}

static int check(int64_t rt, int64_t tn, int cl, int grid, bool waits)
{
    const HandOut h = hand_out(rt, tn, cl, grid, waits);
    auto total_of = [&](int x) { return (int)resident_list_tiles(rt, tn, x, cl); };
    int64_t draws = 0, all = 0;
    for (int x = 0; x < kTicketLists; ++x) { draws += resident_list_draws(total_of(x), grid, x, h); all += total_of(x); }
    if (all != rt * tn) return bad("lists", rt, tn, cl, grid);
    if (all <= grid ? !h.by_rank : all > (int64_t)kStaticRounds * grid ? h.by_rank : !waits && !h.by_rank) return bad("by rank", rt, tn, cl, grid);
    if (!h.by_rank) return h.rounds >= 1 && draws > 0 ? 0 : bad("draws", rt, tn, cl, grid);
    if (draws) return bad("draws by rank", rt, tn, cl, grid);
    for (int x = 0; x < kTicketLists; ++x)       // a tile that waits for its piece holds up no second one from another list
        if (waits && h.rounds > 1 && total_of(x) > h.rounds * resident_list_homes(grid, x)) return bad("uneven", rt, tn, cl, grid);
    std::vector<std::vector<int>> seen(kTicketLists);
    for (int x = 0; x < kTicketLists; ++x) seen[x].assign(total_of(x), 0);
    int64_t n = 0;
    for (int b = 0; b < grid; ++b) {
        bool more = true;
        for (int taken = 0; taken < h.rounds; ++taken) {
            int x = -1, t = -1;
            const bool got = tile_by_rank(b % kTicketLists, b / kTicketLists, taken, grid, h.rounds, total_of, x, t);
            if (got && (!more || x < 0 || x >= kTicketLists || t < 0 || t >= total_of(x) || seen[x][t]++)) return bad("taken", rt, tn, cl, grid);
            more = got;
            n += got;
        }
    }
    return n == all ? 0 : bad("left over", rt, tn, cl, grid);
}

int main()
{
    int n = 0;
    for (int cl = 1; cl <= 8; cl *= 2)
        for (int64_t tn : {1, 2, 3, 5, 8, 12, 24, 28, 58})
            for (int64_t rt : {1, 2, 7, 8, 9, 21, 22, 45, 58, 64, 84, 300}) {
                if (cl > tn) continue;
                for (int slots : {1, 5, 8, 248, 256, 512}) {
                    const int grid = (int)(rt * tn < slots ? rt * tn : slots);
                    if (check(rt, tn, cl, grid, false) || check(rt, tn, cl, grid, true)) return 1;
                    n += 2;
                }
            }
    printf("%d launches\n", n);
    return 0;
}
"""


def test_every_tile_is_handed_out_once(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    src, exe = tmp_path / "hand_out.hip", tmp_path / "hand_out"
    src.write_text(PROGRAM)
    r = subprocess.run([hipcc, "-O1", "-std=c++17", "--offload-host-only", "-I", _build.CSRC, str(src), "-o", str(exe)],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-2000:]
    r = subprocess.run([str(exe)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout
    assert int(r.stdout.split()[0]) > 1000
