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

// ---- one launch for the selection and the union, or several ----

constexpr int kLseThreads = 1024;   // of the workgroup that a subgraph has in the one launch

// Short segments whose union the launches over the whole device form sooner than one workgroup per subgraph does.
// Long ones, of 32 keys a thread, where most are long or there are few: the one launch is as long as its longest segment, the others
// take longer for every subgraph and member (four steps; one 17,000 and m - 1 of 1,500 of a GEMM: m = 32, k = 64, 6 % less in several
// launches, k = 512 4 %, m = 128 7 and 51 % more; 24,000, k = 512: m = 32 8 % less, m = 64 5 % more; 32,768: m = 64 as long; 1,000 of 300
// beside a 17,000, k = 8: 516 us in one, 722 in several; 128 x 32,768, k = 64, 34 % less).
// And those whose S_spec has an old and a new member for every thread, where k is not just above half the threads' number or the
// segments are not as short (k = 1,024 of 1,024: 142 -> 133 us, of 4,000 149 -> 133; k = 600 of 600 124 -> 128, of 4,000 5 % less).
// Not where members are many: each subgraph has a compute unit to itself in the one launch, and shares the others with all
// (50 x 20,000, k = 512: 376 in one, 395 in several; 20 x 4,000, k = 1,000: 196 and 207).
constexpr int64_t kSpreadMembers = 20480, kSpreadPairs = 4096, kShortPairs = 1536;
constexpr bool spread_out(int64_t n, int64_t longest, int32_t n_sg, int32_t k)
{
    const int64_t members = (int64_t)n_sg * k, many_keys = 16 * kLseThreads;
    if (longest > many_keys && members <= kSpreadMembers && (n > n_sg * many_keys || 2 * n_sg * (k + 512ll) <= 5 * longest)) return true;
    return k > kLseThreads / 2 && members <= kSpreadPairs && (k >= 704 || longest > kShortPairs);
}

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
// Where not every segment of a call has a table, the launches that make children remain, each as long as it takes for its other segments, and
// the table's launch is paid for by one segment at least that has more children per entry (four steps of 20 x 60,000 of an encoder layer, k = 264,
// tables of the plain products at 4.2 and none of the batched ones: 277 us without, 285 with; 6 x 200,000, k = 740, at 5 288 and 293;
// four classes of 300,000, k = 793, tables at 7, 4.9 and none 432 and 420).
constexpr int64_t kPartialGain = 6;

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

// Drops the tables of a call that has segments without one, unless they pay; entries[s]: of the table of segment s, 0 where there is none.
inline void drop_partial(const int64_t* seg_off, int32_t n_sg, int64_t* entries)
{
    bool pay = true;
    for (int32_t s = 0; s < n_sg; ++s) pay = pay && entries[s] > 0;
    for (int32_t s = 0; s < n_sg; ++s) pay = pay || (entries[s] > 0 && seg_off[s + 1] - seg_off[s] >= kPartialGain * entries[s]);
    for (int32_t s = 0; s < n_sg; ++s) entries[s] = pay ? entries[s] : 0;
}

}  // namespace pruner
