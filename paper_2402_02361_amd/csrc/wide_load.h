// Where the draft kernel reads: plain C++, so that the rule can be checked on the host over every size.
#pragma once
#include <stdint.h>

namespace pruner {

// Candidates per thread where loads are wide: four, if the population holds that many.
constexpr int load_width(int64_t n) { return n >= 4 ? 4 : 1; }

// The first of the VEC neighbouring candidates that the thread of candidate c reads from every row: c itself, or the last place from
// which VEC candidates still lie in the population.  (Its end, not the row's: what lies between the population and the pitch
// need not be memory of the caller's, the last row of a window at the right edge of a wider matrix ends with the window.)
template <int VEC> constexpr int64_t load_begin(int64_t c, int64_t n) { return c + VEC <= n ? c : n - VEC; }

}  // namespace pruner
