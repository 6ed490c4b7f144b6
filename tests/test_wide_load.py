"""Which elements the draft kernel's threads read, on the host: every candidate is covered and nothing behind the population is
read, also where the population is a window at the right edge of a wider matrix.  And which maxima a selection by blocks reads, where
every block of a level is chosen (a bound of 0): none behind a segment's and the three words that the workspace has there."""
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


LEVELS = r"""
#include "wide_load.h"
#include <cstdio>
// the last blocks of a level, as chosen by threads of `of` quads each, and the last parts of these on the levels below
static int check(int len)
{
    const int level[3] = {(len + 15) >> 4, (len + 63) >> 6, (len + 255) >> 8};
    for (int top = 0; top < 3; ++top)
        for (int of = 1; of <= 4; ++of) {
            const int n = level[top], n_quads = (n + 3) >> 2, q0 = (n_quads - 1) / of * of, mine = n_quads - q0;
            int last = -1, from = n;   // the last chosen block, the first that is looked at
            const uint32_t held = pruner::maxima_held(mine, 4 * (n_quads - 1), n);
            for (int j = 0; j < 16; ++j)
                if (held >> j & 1) last = 4 * q0 + j, from = from < last ? from : last;
            if (last != n - 1 || from != 4 * q0) return std::printf("%d entries, level %d, %d quads: %d to %d of %d\n", len, top, of, from, last, n), 1;
            for (int below = top - 1; below >= 0; --below) {
                const int first = 4 * last;
                if (first >= level[below]) return std::printf("%d entries: block %d of level %d has no parts\n", len, last, below + 1), 1;
                if (first + 4 > level[below] + 3) return std::printf("%d entries: read up to %d of %d\n", len, first + 4, level[below]), 1;
                const uint32_t parts = pruner::maxima_held(1, first, level[below]);
                for (int j = 0; j < 16; ++j)
                    if (parts >> j & 1) last = first + j;
                if (last != level[below] - 1) return std::printf("%d entries: last part %d of %d\n", len, last, level[below]), 1;
            }
            // a thread behind the last quad
            if (pruner::maxima_held(0, 4 * (n_quads - 1), n) != 0 || pruner::maxima_held(-3, 4 * (n_quads - 1), n) != 0) return 1;
        }
    return 0;
}
int main()
{
    for (int len = 16385; len < 16385 + 1100; ++len)
        if (check(len) || check(len + (1 << 18)) || check(len + (1 << 20)) || check((1 << 22) - len)) return 1;
    return 0;
}
"""


def test_no_block_behind_the_last_is_chosen(tmp_path):
    src, exe = tmp_path / "levels.cpp", tmp_path / "levels"
    src.write_text(LEVELS)
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "paper_2402_02361_amd", "csrc"), str(src), "-o", str(exe)])
    run = subprocess.run([str(exe)], capture_output=True, text=True)
    assert run.returncode == 0, run.stdout
