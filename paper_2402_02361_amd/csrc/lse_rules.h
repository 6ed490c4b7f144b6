// Which parts of the explorer loop take which route: plain C++, so that the rules can be checked on the host.
#pragma once
#include <stdint.h>

#include "pruner.h"

namespace pruner {

// One class (two where the kernels make their candidates) and few candidates: a launch takes them one to a thread, on four times the
// compute units, a thread's chain of divisions a quarter as long (reading: 4,096 GEMM candidates 5.8 -> 5.0 us, 65,536 of a
// convolution 7.4 -> 5.8, 262,144 7.7 -> 7.0; making: 8,000 10.6 -> 5.6, 65,536 13.2 -> 7.7, 262,144 13.8 -> 11.8; at 400,000 a tenth
// less as well, but the maxima of 256 neighbours want fours).
constexpr int64_t kSpreadMax = 1 << 18;
constexpr bool one_each(int64_t n, int n_classes, bool makes, bool wants_fours) { return n <= kSpreadMax && n_classes <= (makes ? 2 : 1) && !wants_fours; }

// ---- the table of all children that a subgraph's S_spec can have (lse_child.h numbers them) ----

// Moves of a schedule: a source and a destination among the levels of an axis, and the plain copy.
constexpr int move_count(int n_sp, int n_rd, int rd_levels) { return 12 * n_sp + rd_levels * (rd_levels - 1) * n_rd + 1; }

// The values of a move's prime draw that matter for a subgraph's schedules (1, 2 or 4; 0: more than a table tells apart): their factors
// divide the extents.
inline int told_apart(const pruner_subgraph& s)
{
    int most = 0;
    for (int a = 0; a < s.n_sp + s.n_rd; ++a) {
        int primes = 0;
        int32_t rest = s.extent[a];
        for (int32_t p = 2; p * p <= rest; ++p) {
            if (rest % p == 0) ++primes;
            while (rest % p == 0) rest /= p;
        }
        if (rest > 1) ++primes;
        most = primes > most ? primes : most;
    }
    return s.rd_levels < 2 ? 0 : most <= 1 ? 1 : most == 2 ? 2 : most == 3 ? 4 : 0;
}

// Children per entry of a table from which one is made: an entry is made and scored as a child is without a table, a child with one costs a
// fifth of that and a line from the vector cache, and the table is a launch more.
constexpr int64_t kTableGain = 4;

// Not where children are made one to a thread: that launch is bound by latency, looking up is no shorter a chain, and the table is a launch
// before it (four steps of a GEMM's 33,000 136 us without a table, 147 with; 65,536 142 and 154; 262,144 161 and 171; two classes of
// 100,000 180 and 184; a convolution's 262,144 179 and 182.  Of four children to a thread, 300,000: 181 and 178, a convolution's 199 and
// 190; of three classes of 50,000, whose children would be a launch's and read again, 200 and 188).
constexpr bool table_pays(int64_t n, int n_classes, bool wants_fours) { return !one_each(n, n_classes, true, wants_fours); }

// Entries of the table of a segment of `len` children, a multiple of four (0: none is made), and the values told apart in them.  Extents are
// factorised only where the segment is long enough for any table: 1,000 subgraphs of extents with large primes and 1,100 children each were
// 0.8 ms of host time in a call of 2 ms.
inline int64_t table_entries(const pruner_subgraph& s, int64_t len, int32_t k, int* draws)
{
    auto entries = [&](int of_a_move) { return ((int64_t)k * of_a_move * move_count(s.n_sp, s.n_rd, s.rd_levels) + 3) & ~3ll; };
    *draws = 0;
    if (len < kTableGain * entries(1)) return 0;
    *draws = told_apart(s);
    return *draws > 0 && len >= kTableGain * entries(*draws) ? entries(*draws) : 0;
}

}  // namespace pruner
