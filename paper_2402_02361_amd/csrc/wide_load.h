// Where the draft kernel reads, and which of a level's maxima a selection reads: plain C++, so that the rules can be checked on the
// host over every size.
#pragma once
#include <stdint.h>

namespace pruner {

// Candidates per thread where loads are wide: four, if the population holds that many.
constexpr int load_width(int64_t n) { return n >= 4 ? 4 : 1; }

// The first of the VEC neighbouring candidates that the thread of candidate c reads from every row: c itself, or the last place from
// which VEC candidates still lie in the population.  (Its end, not the row's: what lies between the population and the pitch
// need not be memory of the caller's, the last row of a window at the right edge of a wider matrix ends with the window.)
template <int VEC> constexpr int64_t load_begin(int64_t c, int64_t n) { return c + VEC <= n ? c : n - VEC; }

// The maxima that `quads` neighbouring quads of a level of n hold, a bit each: all four but for the last quad, which begins at
// number `first_of_last` and may reach past the end.  What lies there is no block: named as one, its parts on the next level would be
// read behind the end of that level.
constexpr uint32_t maxima_held(int quads, int first_of_last, int n)
{
    return quads < 1 ? 0u : (1u << (4 * (quads - 1) + (n - first_of_last < 4 ? n - first_of_last : 4))) - 1u;
}

}  // namespace pruner
