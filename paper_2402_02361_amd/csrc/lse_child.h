// The mutation of Alg. 2's SchMutation as a device function, for the kernel that mutates a population in place and for
// the draft kernel that produces and scores the children in one pass.
#pragma once
#include "common.h"
#include "lse_rules.h"

namespace pruner {

struct alignas(8) LseSeg {
    int64_t begin, end;
    int32_t n_sp, n_rd, rd_levels, n_slots;
    int32_t frag[3];     // 0 outside fragment mode
    uint32_t table;      // where the subgraph's entries of the table of all possible children begin, a multiple of four, and how many values of a
                         // move's prime draw it tells apart in the low bits (table_word() below; those 0: no table)
};

// A member of S_spec as one record: its tile factors side by side (32 x uint16 = 64 bytes), so that a parent is read
// with a few 16-byte loads instead of one load per factor.
constexpr int kAosSlots = 32;
static_assert(PRUNER_MAX_SLOTS <= kAosSlots, "a schedule fits one 64-byte record");

// SplitMix64's output function on a state z = seed + c * gamma.
constexpr uint64_t kGamma = 0x9E3779B97F4A7C15ull;
__device__ __forceinline__ uint64_t splitmix64_mix(uint64_t z)
{
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}
// floor(x * n / 256) for an 8-bit field x and n < 2^16: one full-rate multiply
__device__ __forceinline__ int pick8(uint32_t x, uint32_t n) { return (int)(__umul24(x & 0xFFu, n) >> 8); }

// Whether p divides x, for 0 < p, x < 2^16; q is then x / p.  x * (1/p) in binary32 is off by less than 0.03 from the
// true quotient, so rounding gives the quotient exactly when there is one, and q * p == x holds for no q otherwise.
__device__ __forceinline__ bool divides(uint32_t p, uint32_t x, uint32_t& q)
{
    q = (uint32_t)__builtin_rintf((float)x * __builtin_amdgcn_rcpf((float)p));
    return __umul24(q, p) == x;
}

constexpr int kAosWords = kAosSlots / 2;

// What the draws of a child decide: its parent, and whether and how one of the parent's tile factors gives a prime factor to another level.
struct Move {
    int parent;            // the member of S_spec
    bool moves;            // else the child is a plain copy
    int axis, src, dst;    // dst: the destination among the other levels of the axis, 0 .. levels - 2
    uint32_t prime_draw;   // eight bits that pick one of the distinct primes of the factor
};

__device__ __forceinline__ int levels_of(const LseSeg& seg, int axis) { return axis < seg.n_sp ? 4 : seg.rd_levels; }

// The first draw of a child, and (from its generator state z1) what the second decides; count: members of S_spec.
__device__ __forceinline__ void drawn_parent(uint64_t z1, int count, uint32_t mutate_q16, Move& m)
{
    const uint64_t u1 = splitmix64_mix(z1);
    m.parent = (int)__umulhi((uint32_t)u1, (uint32_t)count);
    m.moves = ((uint32_t)(u1 >> 32) & 0xFFFFu) < mutate_q16;
}
__device__ __forceinline__ void drawn_move(const LseSeg& seg, uint64_t z1, Move& m)
{
    const uint32_t u2 = (uint32_t)splitmix64_mix(z1 + kGamma);
    m.axis = pick8(u2, (uint32_t)(seg.n_sp + seg.n_rd));
    const int levels = levels_of(seg, m.axis);
    m.src = pick8(u2 >> 8, (uint32_t)levels);
    m.dst = pick8(u2 >> 16, (uint32_t)(levels - 1));
    m.prime_draw = u2 >> 24;
}

// ---- all possible children of a parent ----
// A subgraph's moves are numbered by axis, source and destination, the plain copy last; every move has as many entries as its
// prime draw has distinguishable values: one where a factor has one distinct prime at most, two halves for two, and the four pieces
// that halves and thirds cut 0..255 into for three.  Subgraphs with more primes in an extent have no table.
__host__ __device__ constexpr int primes_told_apart(int draws) { return draws == 4 ? 3 : draws; }
// LseSeg::table: one, two or four values are 1, 2, 3 in the two low bits
__host__ __device__ constexpr uint32_t table_word(uint32_t at, int draws) { return at | (draws == 4 ? 3u : (uint32_t)draws); }
__host__ __device__ constexpr int draws_of(const LseSeg& seg) { return (int)((1u << (seg.table & 3u)) >> 1); }
__host__ __device__ constexpr uint32_t table_at(const LseSeg& seg) { return seg.table & ~3u; }
__host__ __device__ constexpr int entries_per_parent(const LseSeg& seg) { return draws_of(seg) * move_count(seg.n_sp, seg.n_rd, seg.rd_levels); }

struct MoveNumbers {   // a subgraph's constants, the same for the whole wavefront
    uint32_t n_sp, n_axes, rd_levels, per_parent, plain_copy, count;
};
template <int DRAWS> __device__ __forceinline__ MoveNumbers move_numbers(const LseSeg& seg, int count)
{
    MoveNumbers m;
    m.n_sp = (uint32_t)__builtin_amdgcn_readfirstlane(seg.n_sp);
    m.n_axes = (uint32_t)__builtin_amdgcn_readfirstlane(seg.n_sp + seg.n_rd);
    m.rd_levels = (uint32_t)__builtin_amdgcn_readfirstlane(seg.rd_levels);
    m.plain_copy = (uint32_t)move_count((int)m.n_sp, (int)(m.n_axes - m.n_sp), (int)m.rd_levels) - 1u;
    m.per_parent = DRAWS * (m.plain_copy + 1u);
    m.count = (uint32_t)__builtin_amdgcn_readfirstlane(count);
    return m;
}
// The entry of the child whose first draw has the generator state z1 (drawn_move(), numbered), from the subgraph's first on.
template <int DRAWS> __device__ __forceinline__ uint32_t variant_drawn(const MoveNumbers& m, uint64_t z1, uint32_t mutate_q16)
{
    const uint64_t u1 = splitmix64_mix(z1);
    const uint32_t u2 = (uint32_t)splitmix64_mix(z1 + kGamma);
    const uint32_t parent = __umulhi((uint32_t)u1, m.count);
    const bool moves = ((uint32_t)(u1 >> 32) & 0xFFFFu) < mutate_q16;
    const uint32_t axis = (uint32_t)pick8(u2, m.n_axes);
    const bool spatial = axis < m.n_sp;
    const uint32_t others = spatial ? 3u : m.rd_levels - 1u, each = spatial ? 12u : m.rd_levels * (m.rd_levels - 1u), from = spatial ? 0u : m.n_sp * (12u - m.rd_levels * (m.rd_levels - 1u));
    const uint32_t src = (uint32_t)pick8(u2 >> 8, others + 1u), dst = (uint32_t)pick8(u2 >> 16, others), x = u2 >> 24;
    const uint32_t number = moves ? __umul24(axis, each) + from + __umul24(src, others) + dst : m.plain_copy;
    const uint32_t piece = DRAWS == 1 ? 0u : DRAWS == 2 ? x >> 7 : (x >= 86u ? 1u : 0u) + (x >= 128u ? 1u : 0u) + (x >= 171u ? 1u : 0u);
    return __umul24(parent, m.per_parent) + number * DRAWS + piece;
}
__device__ __forceinline__ Move move_of_variant(const LseSeg& seg, int variant)   // the other way round
{
    Move m{};
    const int draws = draws_of(seg), per_parent = entries_per_parent(seg);
    m.parent = variant / per_parent;
    const int left = variant - m.parent * per_parent, number = left / draws, piece = left - number * draws;
    m.moves = number + 1 < move_count(seg.n_sp, seg.n_rd, seg.rd_levels);
    const bool spatial = number < 12 * seg.n_sp;
    const int levels = spatial ? 4 : seg.rd_levels, each = levels * (levels - 1), in = spatial ? number : number - 12 * seg.n_sp;
    m.axis = m.moves ? (spatial ? 0 : seg.n_sp) + in / each : 0;
    m.src = m.moves ? in % each / (levels - 1) : 0;
    m.dst = m.moves ? in % each % (levels - 1) : 0;
    m.prime_draw = draws == 1 ? 0u : draws == 2 ? (uint32_t)piece << 7 : piece == 0 ? 0u : piece == 1 ? 86u : piece == 2 ? 128u : 171u;
    return m;
}

// The child of subgraph `sub` that a move makes (rest_of(m) says the rest of a move that is one, while the parent's record is on its way):
// `packed` receives its tile factors, two per word, as the record holds them.
// The two slots a mutation touches are read from the record directly, and the child differs from the record by XOR
// masks on their two words: no slot is looked up in registers by a computed index.  Returns the number of distinct primes among
// which the draw picked (0 for a plain copy).
template <int NP, class Rest>   // NP: the 16-byte pieces of a record that the subgraph's slots reach; words past them stay 0
__device__ __forceinline__ int child_of_move(const LseSeg& seg, int sub, int k, Move m, const uint4* __restrict__ spec_aos, uint32_t (&packed)[kAosWords], Rest&& rest_of)
{
    const uint4* parent = spec_aos + ((int64_t)sub * k + (int64_t)m.parent) * (kAosSlots / 8);
#pragma unroll
    for (int q = 0; q < kAosSlots / 8; ++q) {
        uint4 w4 = make_uint4(0u, 0u, 0u, 0u);
        if (q < NP) w4 = parent[q];
        packed[4 * q] = w4.x, packed[4 * q + 1] = w4.y, packed[4 * q + 2] = w4.z, packed[4 * q + 3] = w4.w;
    }
    int word_src = -1, word_dst = -1;
    uint32_t mask_src = 0, mask_dst = 0;
    int n_primes = 0;
    if (m.moves) {
        rest_of(m);
        const int n_axes = seg.n_sp + seg.n_rd, axis = m.axis, levels = levels_of(seg, axis), src = m.src;
        const int base = axis < seg.n_sp ? axis * 4 : seg.n_sp * 4 + (axis - seg.n_sp) * seg.rd_levels;
        const int dst = m.dst >= src ? m.dst + 1 : m.dst;
        const uint16_t* slots = reinterpret_cast<const uint16_t*>(parent);
        const uint32_t v = slots[base + src], at_dst_value = slots[base + dst];
        // distinct prime factors of v in ascending order (at most six below 2^16), 16 bits each, the last found lowest
        uint64_t primes_lo = 0;
        uint32_t primes_hi = 0;
        uint32_t rest = v;
        if (rest > 1 && (rest & 1u) == 0) {   // the factor 2 by shifts: tile factors are mostly powers of two
            primes_lo = 2, n_primes = 1;
            rest >>= __builtin_ctz(rest);
        }
        for (uint32_t p = 3; p * p <= rest; p += 2) {
            uint32_t q;
            if (divides(p, rest, q)) {
                primes_hi = (primes_hi << 16) | (uint32_t)(primes_lo >> 48), primes_lo = (primes_lo << 16) | p, ++n_primes;
                do rest = q; while (divides(p, rest, q));
            }
        }
        if (rest > 1) primes_hi = (primes_hi << 16) | (uint32_t)(primes_lo >> 48), primes_lo = (primes_lo << 16) | rest, ++n_primes;
        if (n_primes > 0) {
            const int back = n_primes - 1 - pick8(m.prime_draw, (uint32_t)n_primes);   // the draw picks one of them
            const uint32_t p = (back < 4 ? (uint32_t)(primes_lo >> (16 * (back & 3))) : primes_hi >> (16 * (back & 1))) & 0xFFFFu;
            uint32_t smaller = v >> 1;
            if (p != 2) divides(p, v, smaller);
            bool ok = true;
            if (seg.frag[0] > 0 && src == levels - 1) {
                int frag = 0;
                if (axis == seg.n_sp - 2) frag = seg.frag[0];
                if (axis == seg.n_sp - 1) frag = seg.frag[1];
                if (axis == n_axes - 1) frag = seg.frag[2];
                uint32_t q;
                if (frag > 0 && ((frag & (frag - 1)) == 0 ? (smaller & (uint32_t)(frag - 1)) != 0 : frag > 0xFFFF || !divides((uint32_t)frag, smaller, q)))
                    ok = false;
            }
            if (ok) {
                const int at_src = base + src, at_dst = base + dst;
                word_src = at_src >> 1, word_dst = at_dst >> 1;
                mask_src = ((smaller ^ v) & 0xFFFFu) << (16 * (at_src & 1));
                mask_dst = (((at_dst_value * p) ^ at_dst_value) & 0xFFFFu) << (16 * (at_dst & 1));
            }
        }
    }
#pragma unroll
    for (int w = 0; w < 4 * NP; ++w) packed[w] ^= (w == word_src ? mask_src : 0u) ^ (w == word_dst ? mask_dst : 0u);
    return n_primes;
}

// One child of subgraph `sub` (its S_spec holds `count` >= 1 schedules) from the generator state z1 of its first draw.
template <int NP>
__device__ __forceinline__ void lse_child(const LseSeg& seg, int sub, int count, int k, uint64_t z1, const uint4* __restrict__ spec_aos,
                                          uint32_t mutate_q16, uint32_t (&packed)[kAosWords])
{
    Move m;
    drawn_parent(z1, count, mutate_q16, m);
    (void)child_of_move<NP>(seg, sub, k, m, spec_aos, packed, [&](Move& its) { drawn_move(seg, z1, its); });
}

// The generator state of child j's first draw in step `step`: child j draws outputs c + 1 and c + 2, c = step * 2^41 + 2 j.
__device__ __forceinline__ uint64_t lse_child_state(uint64_t seed, uint64_t step, int64_t j) { return seed + ((step << 41) + 2 * (uint64_t)j + 1) * kGamma; }

// What the mutation reads beside the segment table.
struct MutArgs {
    const LseSeg* segs;        // by subgraph
    const uint4* spec_aos;     // S_spec as records, [n_sg * k][kAosSlots / 8]
    const int32_t* spec_count; // members per subgraph
    uint64_t seed, step;
    uint32_t mutate_q16;
    int32_t k;
    uint4* child_aos;          // the children as records too, [n][kAosSlots / 8] (the pieces their slots reach); or null
    const float* table;        // the scores of all possible children (LseSeg::table); or null: every child is made and scored
    int32_t* odd;              // by subgraph: not 0 where a schedule of S_spec has more primes than the table tells apart (it is then not used)
    int32_t variants;          // the launch makes and scores, instead of children, the table's entries
};

}  // namespace pruner
