"""The rules of the explorer loop's routes, on the host: which segments get a table of all their children, and that asking costs nothing
where the answer is no."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

COMMON = r"""
#include "lse_rules.h"
#include <chrono>
#include <cstdio>
#include <vector>
static pruner_subgraph gemm(int m, int n, int k)
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
        bad += pruner::told_apart(gemm(210, 64, 32)) != 0 || pruner::told_apart(gemm(64, 64, 30030)) != 0;
    }
    return bad;
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


@pytest.mark.parametrize("program", [ENTRIES, TIME], ids=["entries", "time"])
def test_table_rule(tmp_path, program):
    src, exe = tmp_path / "rules.cpp", tmp_path / "rules"
    src.write_text(COMMON + program)
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-Wall", "-I", os.path.join(ROOT, "paper_2402_02361_amd", "csrc"), "-I", os.path.join(ROOT, "include"), str(src), "-o", str(exe)])
    run = subprocess.run([str(exe)], capture_output=True, text=True)
    assert run.returncode == 0, run.stdout
