"""The rules of the explorer loop's routes, on the host: which segments get a table of all their children, that asking costs nothing where the
answer is no, and which short segments leave the one launch."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

COMMON = r"""
#include "lse_rules.h"
#include <chrono>
#include <cstdio>
#include <vector>
[[maybe_unused]] static pruner_subgraph gemm(int m, int n, int k)
{
    pruner_subgraph s{};
    s.n_sp = 2, s.n_rd = 1, s.rd_levels = 2;
    s.extent[0] = m, s.extent[1] = n, s.extent[2] = k;
    return s;
}
"""

ENTRIES = r"""
static int check(pruner_subgraph s, int values, int k)
{
    const int64_t entries = ((int64_t)k * values * 27 + 3) / 4 * 4;   // 2 x 12 and 2 moves, and the plain copy
    int draws = -1;
    if (pruner::told_apart(s) != values) return std::printf("%d x %d x %d\n", s.extent[0], s.extent[1], s.extent[2]), 1;
    const int64_t at = pruner::table_entries(s, 4 * entries, k, &draws);
    if (values ? at != entries || draws != values : at != 0) return std::printf("k %d: %ld entries\n", k, (long)at), 1;
    return pruner::table_entries(s, 4 * entries - 1, k, &draws) != 0;
}
int main()
{
    int bad = 0;
    // where children are made one to a thread they are not looked up
    bad += pruner::table_pays(33000, 1, false) || pruner::table_pays(1 << 18, 1, false) || pruner::table_pays(1 << 18, 2, false);
    bad += !pruner::table_pays((1 << 18) + 1, 1, false) || !pruner::table_pays(100000, 3, false) || !pruner::table_pays(100000, 1, true);
    for (int k : {1, 17, 512, 4096}) {
        bad += check(gemm(64, 1, 65536 / 2), 1, k) + check(gemm(97, 13, 25), 1, k) + check(gemm(96, 80, 72), 2, k) + check(gemm(60, 90, 64), 4, k);
        // five children per entry are enough where all segments have a table, or one of them has six
        const int64_t e = ((int64_t)k * 2 * 27 + 3) / 4 * 4, off[4] = {0, 5 * e, 10 * e, 16 * e};
        for (int kept : {0, 1, 2, 3, 4, 5, 6, 7}) {
            int64_t entries[3] = {kept & 1 ? e : 0, kept & 2 ? e : 0, kept & 4 ? e : 0};
            pruner::drop_partial(off, 3, entries);
            for (int s = 0; s < 3; ++s) bad += entries[s] != (kept >> s & 1 && kept & 4 ? e : 0);
            if (kept != 3) continue;
            int64_t two[2] = {e, e};
            pruner::drop_partial(off, 2, two);
            bad += two[0] != e || two[1] != e;
        }
        bad += pruner::told_apart(gemm(210, 64, 32)) != 0 || pruner::told_apart(gemm(64, 64, 30030)) != 0;
    }
    return bad;
}
"""

# the routes that were the faster ones, by a GEMM's, an encoder's and four classes' subgraphs together
ROUTES = r"""
int main()
{
    int bad = 0;
    auto several = [&](int64_t longest, int n_sg, int64_t others, int k, bool want) {
        if (pruner::spread_out(longest + (n_sg - 1) * others, longest, n_sg, k) != want) bad += std::printf("%ld, %d subgraphs of %ld, k %d\n", (long)longest, n_sg, (long)others, k);
    };
    for (int k : {1, 8, 64, 512}) several(16384, 1, 0, k, false), several(32768, 1, 0, k, true), several(24000, 16, 1500, k, true);
    for (int m : {301, 1001, 2501}) several(17000, m, 300, 8, false);
    for (int k : {16, 64, 256}) several(17000, 128, 1500, k, false), several(17000, 32, 1500, k, true);
    several(17000, 64, 1500, 256, false), several(17000, 64, 1500, 512, false), several(24000, 64, 1500, 64, true), several(24000, 128, 1500, 256, false);
    several(24000, 64, 1500, 512, false), several(32768, 64, 1500, 256, true), several(32768, 128, 1500, 512, false), several(32000, 101, 1500, 64, true);
    several(32768, 128, 32768, 64, true), several(32768, 300, 32768, 64, true), several(24000, 64, 24000, 256, true), several(20000, 50, 20000, 512, false);
    several(520, 1, 0, 513, false), several(600, 1, 0, 600, false), several(1000, 7, 1000, 513, false), several(1100, 7, 1100, 600, false);
    several(1000, 1, 0, 1000, true), several(1024, 4, 1024, 1024, true), several(720, 1, 0, 704, true), several(2000, 7, 2000, 585, true), several(8000, 7, 8000, 520, true);
    several(4000, 20, 4000, 1000, false), several(4000, 1, 0, 512, false);
    return bad != 0;
}
"""

# the largest primes that three axes may have, a thousand subgraphs: for segments that are too short, and for long ones
TIME = r"""
static double seconds(int64_t len)
{
    std::vector<pruner_subgraph> all;
    for (int p : {46337, 46327, 46309, 46307, 46301}) all.push_back(gemm(p, 40009, 65521));
    double best = 1e9;
    for (int rep = 0; rep < 20; ++rep) {
        const auto from = std::chrono::steady_clock::now();
        int64_t sum = 0;
        for (int s = 0; s < 1000; ++s) {
            int draws;
            sum += pruner::table_entries(all[s % 5], len, 1025, &draws);
        }
        const double t = std::chrono::duration<double>(std::chrono::steady_clock::now() - from).count();
        if (sum != (len > 200000 ? 27676000 : 0)) return std::printf("%ld entries\n", (long)sum), -1;
        best = t < best ? t : best;
    }
    return best;
}
int main()
{
    const double slow = seconds(300000), fast = seconds(1100);
    std::printf("%g %g\n", slow, fast);
    return slow < 0 || fast < 0 || fast * 10 > slow;
}
"""


@pytest.mark.parametrize("program", [ENTRIES, TIME, ROUTES], ids=["entries", "time", "routes"])
def test_rule(tmp_path, program):
    src, exe = tmp_path / "rules.cpp", tmp_path / "rules"
    src.write_text(COMMON + program)
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-Wall", "-I", os.path.join(ROOT, "paper_2402_02361_amd", "csrc"), "-I", os.path.join(ROOT, "include"), str(src), "-o", str(exe)])
    run = subprocess.run([str(exe)], capture_output=True, text=True)
    assert run.returncode == 0, run.stdout
