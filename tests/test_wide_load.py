"""Which elements the draft kernel's threads read, on the host: every candidate is covered and nothing behind the population is
read, also where the population is a window at the right edge of a wider matrix."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "wide_load.h"
#include <cstdio>
template <int VEC> static int check(int64_t n)
{
    for (int64_t c = 0; c < n; ++c) {   // (segments may begin anywhere, so any candidate can be a thread's first)
        const int64_t at = pruner::load_begin<VEC>(c, n);
        if (at < 0 || at + VEC > n || at > c || c >= at + VEC) return std::printf("n %ld: candidate %ld read from %ld\n", (long)n, (long)c, (long)at), 1;
        // the last row of a window that begins at column 5 of a matrix of two rows of n + 5
        if ((n + 5) + 5 + at + VEC > 2 * (n + 5)) return std::printf("n %ld: past the matrix\n", (long)n), 1;
    }
    return 0;
}
int main()
{
    for (int64_t n = 1; n < 700; ++n)
        if (pruner::load_width(n) == 4 ? check<4>(n) : check<1>(n)) return 1;
    return 0;
}
"""


def test_no_thread_reads_behind_the_population(tmp_path):
    src, exe = tmp_path / "reads.cpp", tmp_path / "reads"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "paper_2402_02361_amd", "csrc"), str(src), "-o", str(exe)])
    run = subprocess.run([str(exe)], capture_output=True, text=True)
    assert run.returncode == 0, run.stdout
