// Device helpers shared by the selection kernels and by the draft kernel when it counts first digits on the fly.
#pragma once
#include "common.h"

#include <type_traits>

namespace pruner {

constexpr int kBins = 2048;   // 11-bit digits

// Larger score <=> larger key; -0.0 and +0.0 share a key.
__device__ __forceinline__ uint32_t key_of(float x)
{
    uint32_t u = __float_as_uint(x);
    if (u == 0x80000000u) u = 0u;
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// The first digit of the selection: a bin of 2048 that grows with the key.  Scores lie within a few dozen octaves, so the bins
// are narrow there: 16 to an octave (four to six per cent of a score) in a window of thirty-four octaves on either side of
// zero (latencies of a tenth of a microsecond and scores in the thousands lie inside), two to an octave outside it.  (With the
// key's upper eleven bits, four bins to an octave, the bin of rank k held thousands of entries; now it holds tens to hundreds,
// and most populations are settled by this digit alone.)  Two more digits of up to eleven bits settle any bin (a bin spans
// 2^19 keys, or 2^22 outside the window).
constexpr uint32_t kFine = 34 * 16;
constexpr uint32_t kWindow = (127 - 23) * 16;   // in units of 1/16 octave: 2^-23
// b = x / 8 below the window, x / 8 + 7/8 of the way into it inside, again x / 8 plus a constant above (x: the magnitude in
// units of 1/16 octave): (x + 7 clamp(x - window, 0, kFine)) / 8, five instructions.  0 .. 987.
__device__ __forceinline__ uint32_t magnitude_bin(uint32_t bits)
{
    const uint32_t x = (bits >> 19) & 0xFFFu;
    int d = (int)x - (int)kWindow;
    d = d > 0 ? d : 0;
    d = d < (int)kFine ? d : (int)kFine;
    return ((uint32_t)__umul24((uint32_t)d, 7u) + x) >> 3;
}
// 1024 + b, or 1023 - b for a negative score
__device__ __forceinline__ uint32_t first_digit_of(uint32_t key)
{
    const uint32_t below_zero = ~(uint32_t)((int32_t)key >> 31);   // all ones for a negative score
    return (magnitude_bin(key ^ below_zero) + 1024u) ^ (below_zero >> 21);
}
// The key and the first digit of a score at once.
__device__ __forceinline__ uint32_t key_and_digit(float score, uint32_t& digit)
{
    uint32_t u = __float_as_uint(score);
    if (u == 0x80000000u) u = 0u;
    const uint32_t below_zero = (uint32_t)((int32_t)u >> 31);
    digit = (magnitude_bin(u) + 1024u) ^ (below_zero >> 21);
    return u ^ (below_zero | 0x80000000u);
}
// The keys of a bin: lowest .. lowest + width.
__device__ __forceinline__ void first_digit_range(uint32_t bin, uint32_t& lowest, uint32_t& width)
{
    static_assert(kWindow % 8 == 0 && kFine % 8 == 0, "bins outside the window are whole");
    const bool negative = bin < 1024u;
    const uint32_t b = negative ? 1023u - bin : bin - 1024u;
    auto begin = [](uint32_t v) { return v < kWindow / 8 ? v * 8 : v < kWindow / 8 + kFine ? kWindow + (v - kWindow / 8) : kWindow + kFine + (v - kWindow / 8 - kFine) * 8; };
    const uint32_t from = begin(b) << 19, to = begin(b + 1) << 19;
    lowest = negative ? 0x80000000u - to : 0x80000000u + from;
    width = to - from - 1u;
}
// The digits after it: the offset from the range's lowest key, its upper eleven bits first.  The shift of that first one.
__device__ __forceinline__ int next_shift(uint32_t width) { const int bits = width ? 32 - __clz(width) : 0; return bits > 11 ? bits - 11 : 0; }

// The score with a given key (every key but the one that -0.0 and +0.0 share belongs to exactly one bit pattern).
constexpr uint32_t kZeroKey = 0x80000000u;
__device__ __forceinline__ float score_of_key(uint32_t key) { return __uint_as_float((key & 0x80000000u) ? (key & 0x7FFFFFFFu) : ~key); }

__device__ __forceinline__ int lane_id() { return __lane_id(); }

// The segment a workgroup belongs to: the last entry of a table sorted by first_block whose first_block is not after
// block b (entry 0 starts at block 0; empty segments share a first block with their successor and are never picked).
// A binary search is a chain of dependent reads, each a round trip to the cache; for tables of up to 256 entries
// every lane reads up to four entries at once instead and the wavefront counts those not after b.  The result is
// the same in every lane.
template <typename Seg> __device__ __forceinline__ int segment_of_block(const Seg* __restrict__ segs, int n_seg, int b)
{
    if (n_seg <= 2) return n_seg == 2 && segs[1].first_block <= b ? 1 : 0;
    if (n_seg <= 4 * kWave) {
        int not_after = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int i = q * kWave + lane_id();
            const bool hit = i < n_seg && segs[i < n_seg ? i : 0].first_block <= b;
            not_after += (int)__popcll(__ballot(hit));
        }
        return not_after - 1;
    }
    int lo = 0, hi = n_seg - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (segs[mid].first_block <= b) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// LDS histogram increment for digits that scatter as a rule: lanes that add to one bin queue on its address, so the lanes that
// share the first active lane's bin are counted with one atomic when they are sixteen or more, everyone else adds 1.  TWICE:
// where they were, so are those that share the bin of the first lane left (sorted scores have two or three bins a
// wavefront: the first digit of 300 sorted segments of 65,536 in 73 us instead of 90; equal ones take 4 us more).
template <bool TWICE = false> __device__ __forceinline__ void light_hist_add(uint32_t* hist, uint32_t digit, bool active)
{
    const unsigned long long there = __ballot(active);
    if (there == 0ull) return;
    const int leader = __ffsll(there) - 1;
    const uint32_t d0 = (uint32_t)__builtin_amdgcn_readlane((int)digit, leader);
    if constexpr (!TWICE) {
        const bool same = active && digit == d0;
        const uint32_t n_same = (uint32_t)__popcll(__ballot(same));
        const bool together = n_same >= 16u;
        if (active && !(together && same)) atomicAdd(&hist[digit], 1u);
        if (together && lane_id() == leader) atomicAdd(&hist[d0], n_same);
    } else {
        const unsigned long long same = __ballot(active && digit == d0);
        const uint32_t n_same = (uint32_t)__popcll(same);
        if (n_same >= 16u) {
            if (lane_id() == leader) atomicAdd(&hist[d0], n_same);
            active = active && digit != d0;
            const unsigned long long rest = there & ~same;
            if (rest != 0ull) {
                const int next = __ffsll(rest) - 1;
                const uint32_t d1 = (uint32_t)__builtin_amdgcn_readlane((int)digit, next);
                const uint32_t n_next = (uint32_t)__popcll(__ballot(active && digit == d1));
                if (n_next >= 16u) {
                    if (lane_id() == next) atomicAdd(&hist[d1], n_next);
                    active = active && digit != d1;
                }
            }
        }
        if (active) atomicAdd(&hist[digit], 1u);
    }
}

// Exclusive prefix sum over the workgroup (NT threads, NT/64 <= 16 wavefronts); all threads must call.
// wave_tot: LDS, 16 entries.  *total receives the workgroup sum.
template <int NT> __device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t* wave_tot, uint32_t* total)
{
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const uint32_t incl = wave_inclusive_sum(v);
    __syncthreads();  // wave_tot may still be read from an earlier call
    if (lane == kWave - 1) wave_tot[wave] = incl;
    __syncthreads();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < NT / kWave; ++w) {
        const uint32_t t = wave_tot[w];
        before += w < wave ? t : 0u;
        all += t;
    }
    *total = all;
    return before + incl - v;
}

// Digit bucket that holds the entry of rank k_rem (ranks counted from the largest digit down) and the rank left
// inside that bucket (out[0], out[1]) and the bucket's population (out[2]).  hist: kBins counters (LDS or global);
// 1024 threads, two bins each.
__device__ __forceinline__ void find_bucket(const uint32_t* hist, uint32_t k_rem, uint32_t* wave_tot, uint32_t* out /* [3] in LDS */)
{
    const int a = kBins - 1 - 2 * (int)threadIdx.x, b = a - 1;
    const uint32_t ha = hist[a], hb = hist[b];
    uint32_t total;
    const uint32_t above = block_excl_scan<kBins / 2>(ha + hb, wave_tot, &total);
    if (above < k_rem && k_rem <= above + ha) {
        out[0] = (uint32_t)a;
        out[1] = k_rem - above;
        out[2] = ha;
    } else if (above + ha < k_rem && k_rem <= above + ha + hb) {
        out[0] = (uint32_t)b;
        out[1] = k_rem - above - ha;
        out[2] = hb;
    }
    __syncthreads();
}

// Merge a workgroup's LDS histogram into its copy of segment s's global histogram ([copies][n_seg][kBins]).
template <int NT>
__device__ __forceinline__ void flush_hist(const uint32_t* hist, uint32_t* __restrict__ ghist, int copies, int n_seg, int s)
{
    uint32_t* mine = ghist + ((int64_t)(blockIdx.x % copies) * n_seg + s) * kBins;
    for (int i = threadIdx.x; i < kBins; i += NT) {
        const uint32_t c = hist[i];
        if (c) atomicAdd(&mine[i], c);
    }
}

// Blocks of 256 neighbouring entries of a segment, counted from the segment's begin: the block whose first entry has the
// global index `first` in segment s keeps its largest key in slot (first >> 8) + s of the block-maximum array.  Slots of
// different blocks differ (inside a segment `first` grows by 256 from block to block; the next segment begins behind
// the last block's first entry and adds one more), so the array needs (n >> 8) + n_seg + 1 words.  The same for blocks of 64.
// Whoever holds the scores in registers (the draft kernel, or a pass of its own) writes them.
__device__ __forceinline__ int64_t block_max_slot(int64_t first, int s) { return (first >> 8) + s; }
__device__ __forceinline__ int64_t block64_slot(int64_t first, int s) { return (first >> 6) + s; }
__device__ __forceinline__ int64_t block16_slot(int64_t first, int s) { return (first >> 4) + s; }

// Leaves the largest keys of the blocks of 16, 64 and 256 neighbours (those that are asked for) that a wavefront
// holds, VEC = 4 or 1 entries per lane, lane 0 at the begin of a block: `top` is the largest key of the lane's own, `first` the index
// of the first of these; entries at or past `end` are none.  The active lanes are 0 .. last.
template <int VEC>
__device__ __forceinline__ void note_maxima(uint32_t top, int64_t first, int last, int64_t end, int s, uint32_t* __restrict__ max16, uint32_t* __restrict__ max64,
                                            uint32_t* __restrict__ max256)
{
    // (a lane whose source is switched off keeps its own)
    const int lane = lane_id(), in_row = lane & 15;
    top = max_with<0x4E, 0xf>(max_with<0xB1, 0xf>(top));   // quad_perm: the neighbour's, the other pair's
    if constexpr (VEC == 4) {
        if (max16 && (lane & 3) == 0 && first < end) max16[block16_slot(first, s)] = top;
        if (!max64 && !max256) return;
        top = max_with<0x118, 0xf>(max_with<0x114, 0xf>(top));   // row_shr:4, row_shr:8: the last lane of a row of 16 has all four
        if (max64 && (in_row == 15 || lane == last) && first - 4 * in_row < end) max64[block64_slot(first - 4 * in_row, s)] = top;
        if (!max256) return;
        top = rows_inclusive_max(top);
        if (lane == last && first - 4 * last < end) max256[block_max_slot(first - 4 * last, s)] = top;
    } else {
        top = max_with<0x118, 0xf>(max_with<0x114, 0xf>(top));
        if (max16 && (in_row == 15 || lane == last) && first - in_row < end) max16[block16_slot(first - in_row, s)] = top;
        if (!max64) return;
        top = rows_inclusive_max(top);
        if (lane == last && first - last < end) max64[block64_slot(first - last, s)] = top;
    }
}

// (key, index) packed so that a larger word is a better entry: key descending, then index ascending.
__device__ __forceinline__ uint64_t compose(uint32_t key, uint32_t gidx) { return ((uint64_t)key << 32) | (uint64_t)(0xFFFFFFFFu - gidx); }
__device__ __forceinline__ uint32_t index_of(uint64_t w) { return 0xFFFFFFFFu - (uint32_t)w; }

// ---- selection of a few entries from a short segment (at most 8192 entries, k at most 64) ------------------------------
//
// The final selection after the verify stage (a few thousand scores per subgraph, a few dozen kept) and small draft
// populations.  No digit passes: an entry is the word (key, index), all words of a segment are distinct, and the k best
// entries are the k largest words.  One workgroup of four wavefronts per segment:
//   1. a thread holds up to 32 words in registers and finds its largest;
//   2. the k-th largest of the 256 thread maxima is a pivot at or below the k-th largest word of the segment (k words,
//      those maxima, are at or above it), and words at or above it can only belong to the k threads whose maxima are:
//      at most 32 k of them, about k on scores in no particular order.  The pivot: every wavefront sorts its 64 maxima
//      across its lanes; a maximum's rank among all 256 is its place in its own wavefront plus, by bisection, the
//      number of larger ones in the other three sorted lists;
//   3. the words at or above the pivot go to a list in LDS; a word's row is the number of larger words in the list.
// 8.7 us for 4,096 entries and k = 64 (10.5 with 32 words per thread and bisections one after the other).

constexpr int kTinyThreads = 256;
constexpr int kTinyPer = 32;   // words per thread, at most
constexpr int kTinyMax = kTinyThreads * kTinyPer;   // 8192 entries per segment
constexpr int kTinyK = 64;
constexpr int kTinyList = kTinyK * kTinyPer;        // words that can reach the pivot

// The word of lane (lane ^ STRIDE).  Inside a row of 16 lanes the data-parallel primitives do it at the vector ALU's own
// rate: a permutation of each group of four lanes for strides 1 and 2, a rotation of the row by 8 for stride 8, and for
// stride 4 the rotation by 12 (which brings lane + 4) or by 4 (lane - 4), whichever the lane needs; across rows the word
// goes through the LDS crossbar.  Every lane of the wavefront must be active.
template <int CTRL> __device__ __forceinline__ uint32_t dpp_move(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, 0xf, 0xf, true);
}
template <int STRIDE> __device__ __forceinline__ uint32_t lane_xor_u32(uint32_t v)
{
    if constexpr (STRIDE == 1) return dpp_move<0xB1>(v);        // quad_perm:[1,0,3,2]
    else if constexpr (STRIDE == 2) return dpp_move<0x4E>(v);   // quad_perm:[2,3,0,1]
    else if constexpr (STRIDE == 4) {
        // both moves run with every lane active (a move whose source lane is switched off reads nothing), then each lane picks
        const uint32_t from_below = dpp_move<0x124>(v), from_above = dpp_move<0x12C>(v);   // row_ror:4 (lane - 4), row_ror:12 (lane + 4)
        return (lane_id() & 4) ? from_below : from_above;
    }
    else if constexpr (STRIDE == 8) return dpp_move<0x128>(v);  // row_ror:8
    else return __shfl_xor(v, STRIDE, kWave);
}
template <int STRIDE> __device__ __forceinline__ uint64_t lane_xor_u64(uint64_t w)
{
    const uint32_t lo = lane_xor_u32<STRIDE>((uint32_t)w), hi = lane_xor_u32<STRIDE>((uint32_t)(w >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// The wavefront's 64 words in descending order over its lanes (bitonic network; partner = lane ^ stride).  Equal words
// (only the all-zero filler) may end up in either order.
__device__ __forceinline__ uint64_t wave_sort_descending(uint64_t w)
{
    const int lane = lane_id();
    auto exchange = [&](auto stride_c, int size) {
        constexpr int stride = decltype(stride_c)::value;
        const uint64_t other = lane_xor_u64<stride>(w);
        const bool lower = (lane & stride) == 0;           // the lower lane of the pair
        const bool down = (lane & size) == 0;              // this merge block is ordered largest first (always, in the last merge)
        w = ((lower == down) == (w > other)) ? w : other;
    };
#pragma unroll
    for (int size = 2; size <= kWave; size <<= 1) {
        if (size >= 64) exchange(std::integral_constant<int, 32>{}, size);
        if (size >= 32) exchange(std::integral_constant<int, 16>{}, size);
        if (size >= 16) exchange(std::integral_constant<int, 8>{}, size);
        if (size >= 8) exchange(std::integral_constant<int, 4>{}, size);
        if (size >= 4) exchange(std::integral_constant<int, 2>{}, size);
        exchange(std::integral_constant<int, 1>{}, size);
    }
    return w;
}

struct TinyLds {
    uint64_t sorted[kTinyThreads / kWave][kWave];   // every wavefront's thread maxima, largest first
    uint64_t pivot_slot;
    uint32_t fill;
    __attribute__((aligned(16))) uint64_t list[kTinyList + 2];
};

// The k best entries of score[seg_begin .. seg_end) as rows idx_out[row * k ..] (and val_out), best first.  A workgroup of
// kTinyThreads threads calls it with all its threads; it begins and ends with everything it read or wrote in L settled
// (callers need no barrier around it except for their own data).  PER: words per thread (at most kTinyThreads PER entries): a word costs
// a dozen instructions whether or not there is an entry for it.
template <int PER>
__device__ __forceinline__ void tiny_select(TinyLds& L, const float* __restrict__ score, int64_t seg_begin, int64_t seg_end, int64_t row, int k,
                                            int32_t* __restrict__ idx_out, float* __restrict__ val_out)
{
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const float* seg_score = score + seg_begin;
    const int len = (int)(seg_end - seg_begin);

    uint64_t w[PER], best = 0;   // 0: no entry (below every word of a number)
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int i = j * kTinyThreads + (int)threadIdx.x;
        w[j] = i < len ? compose(key_of(seg_score[i]), (uint32_t)(seg_begin + i)) : 0ull;
    }
#pragma unroll
    for (int j = 0; j < PER; ++j) best = w[j] > best ? w[j] : best;
    if (threadIdx.x == 0) L.fill = 0;

    const uint64_t mine = wave_sort_descending(best);   // lane p of this wavefront holds its p-th largest maximum
    L.sorted[wave][lane] = mine;
    __syncthreads();
    // rank of `mine` among the 256 maxima = larger ones in this wavefront (lane) + larger ones in the others.  At least k
    // maxima are words of entries (a segment holds at least k entries); the fillers rank behind all of them.  The other lists are
    // searched side by side, in quarters: three looks at each at a time.
    constexpr int kOthers = kTinyThreads / kWave - 1;
    int past[kOthers];
#pragma unroll
    for (int o = 0; o < kOthers; ++o) past[o] = 0;
#pragma unroll
    for (int q = kWave / 4; q >= 1; q >>= 2) {
#pragma unroll
        for (int o = 0; o < kOthers; ++o) {
            const uint64_t* other = L.sorted[(wave + o + 1) % (kTinyThreads / kWave)] + past[o];
            const uint64_t x = other[q - 1], y = other[2 * q - 1], z = other[3 * q - 1];
            past[o] += q * ((x > mine ? 1 : 0) + (y > mine ? 1 : 0) + (z > mine ? 1 : 0));
        }
    }
    static_assert(kWave == 64, "quarters down to one");
    uint32_t rank = (uint32_t)lane;
#pragma unroll
    for (int o = 0; o < kOthers; ++o) rank += (uint32_t)past[o] + (L.sorted[(wave + o + 1) % (kTinyThreads / kWave)][past[o]] > mine ? 1u : 0u);
    if (mine != 0 && rank == (uint32_t)(k - 1)) L.pivot_slot = mine;
    __syncthreads();
    const uint64_t pivot = L.pivot_slot;
    // A thread's words at or above the pivot go to consecutive places of the list: the wavefront's threads share out a
    // range that one of them reserves (one atomic per wavefront, not one per word).
    uint32_t mine_count = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) mine_count += w[j] >= pivot && w[j] != 0 ? 1u : 0u;
    const uint32_t upto = wave_inclusive_sum(mine_count);
    uint32_t wave_base = 0;
    if (lane == kWave - 1 && upto != 0) wave_base = atomicAdd(&L.fill, upto);
    uint32_t at = (uint32_t)__builtin_amdgcn_readlane((int)wave_base, kWave - 1) + upto - mine_count;
    if (mine_count != 0) {
#pragma unroll
        for (int j = 0; j < PER; ++j)
            if (w[j] >= pivot && w[j] != 0) L.list[at++] = w[j];
    }
    __syncthreads();
    const int n_list = (int)L.fill;   // k .. 32 k
    if (threadIdx.x == 0) L.list[n_list] = L.list[n_list + 1] = 0;   // the comparison below reads two words at a time
    __syncthreads();
    typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));
    // four neighbouring lanes to a word, each counting in its own part of the list
    const int part = lane & 3, pairs = (n_list + 1) >> 1;
    for (int e0 = 0; e0 < n_list; e0 += kTinyThreads / 4) {
        const int e = e0 + ((int)threadIdx.x >> 2);
        const uint64_t me = e < n_list ? L.list[e] : ~0ull;
        uint32_t r = 0;
        for (int f = part; f < pairs; f += 4) {
            const u64x2 two = *reinterpret_cast<const u64x2*>(L.list + 2 * f);
            r += two.x > me ? 1u : 0u;
            r += two.y > me ? 1u : 0u;
        }
        r += dpp_move<0xB1>(r);   // quad_perm: the neighbour's, the other pair's
        r += dpp_move<0x4E>(r);
        if (part == 0 && e < n_list && r < (uint32_t)k) {
            const uint32_t gi = index_of(me), kk = (uint32_t)(me >> 32);
            idx_out[row * k + r] = (int32_t)gi;
            // a key names its score, except the one that -0.0 and +0.0 share
            if (val_out) val_out[row * k + r] = kk == kZeroKey ? score[gi] : score_of_key(kk);
        }
    }
    __syncthreads();
}

}  // namespace pruner
