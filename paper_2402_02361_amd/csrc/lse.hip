// Latent Schedule Explorer (Alg. 2) with the population resident on the device:
//   n_steps times { costs = C_SA(S_x);  S_spec = PriorFilter(S_x U S_spec);  S_x = SchMutation(S_x, costs) }.
//
// C_SA and the k best of S_x are the launches of pruner_prior_filter.  The rest of a step:
//   lse_keys    one thread per entry of the union: score key and schedule hash (the k best sit at random places of
//               the population; many workgroups share those reads)
//   lse_merge   one workgroup per subgraph: the union of S_spec and the k best of S_x as a union of SETS (a schedule
//               counts once; identity = score and a 64-bit hash of the tile factors): the order is (score descending,
//               hash ascending, position ascending); the k best of S_x are sorted in LDS, S_spec is in that order
//               already, the two are merged by bisection; copies of a predecessor are dropped, the first k of the
//               rest are the new S_spec
//   lse_copy    the tile factors of the new S_spec, from the old S_spec or from the population; also as one 64-byte
//               record per schedule, from which the mutation reads its parents
//   lse_mutate  one thread per child: a parent drawn uniformly from S_spec (truncation selection: the paper names a
//               genetic algorithm guided by the draft fitness and gives no operator), and with the given probability
//               one prime factor of one tile factor moved to another level of the same axis, fragment multiples kept
// Short segments with a small S_spec (kShortMax entries, k up to kShortK: the populations of an ordinary tuning round) take
// one launch for the selection and all of PriorFilter instead:
//   lse_select  one workgroup per subgraph: the k best of S_x from keys in registers, their schedules' hashes, the union
//               with S_spec and the new S_spec's records
// When the population gets one draft launch per loop-nest class, the mutation of a step is not a launch of its own: the
// next step's draft kernels make the children, store them and score them while they are in registers (the population is
// then written once per step and never read for scoring); only the last step's mutation, whose children nobody scores, is
// a launch.
// Random numbers are counter-based (SplitMix64, Steele/Lea/Flood OOPSLA 2014: draw c is the c-th output of the
// generator started from the seed), so the result does not depend on how the work is laid out.
#include "lse_child.h"
#include "select_common.h"

#include <string.h>

#include <vector>

namespace pruner {
namespace {

constexpr int kLseThreads = 1024;

__device__ __forceinline__ uint64_t splitmix64_draw(uint64_t seed, uint64_t c)
{
    uint64_t z = seed + c * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// identity of a schedule: its own tile slots, in slot order (all slots are requested before the first is hashed)
__device__ __forceinline__ uint64_t schedule_hash(const uint16_t* __restrict__ col, int64_t stride, int n_slots)
{
    uint16_t f[PRUNER_MAX_SLOTS];
#pragma unroll
    for (int r = 0; r < PRUNER_MAX_SLOTS; ++r) f[r] = r < n_slots ? col[r * stride] : (uint16_t)0;
    uint64_t h = (uint64_t)n_slots;
#pragma unroll
    for (int r = 0; r < PRUNER_MAX_SLOTS; ++r)
        if (r < n_slots) h = splitmix64_draw(h, (uint64_t)f[r] + 1);
    return h;
}

__device__ __forceinline__ uint32_t lse_key_of(float x)   // larger score <=> larger key; -0 and +0 share a key
{
    uint32_t u = __float_as_uint(x);
    if (u == 0x80000000u) u = 0u;
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float lse_score_of(uint32_t key) { return __uint_as_float((key & 0x80000000u) ? (key & 0x7FFFFFFFu) : ~key); }

constexpr int32_t kNoSource = (int32_t)0x80000000;

// Entry e of the sort arrays sits at pad(e): one spare entry after every 32, so that threads that walk groups of 8
// neighbouring entries do not all land in the same LDS banks.
__device__ __forceinline__ int pad(int e) { return e + (e >> 5); }
constexpr int padded(int n) { return n + (n >> 5) + 2; }

// 2^LOG entries base + i*s of a bitonic merge of `size`: the strides 2^(LOG-1) s ... s permute them among themselves,
// and they lie in one half of the merge, so they share the direction.
template <int LOG> __device__ __forceinline__ void sort_group(uint64_t* hi, uint64_t* lo, int g, int s, int size)
{
    constexpr int N = 1 << LOG;
    const int base = (g / s) * (N * s) + (g % s);
    const bool down = (base & size) == 0;
    uint64_t xh[N], xl[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        xh[i] = hi[pad(base + i * s)];
        xl[i] = lo[pad(base + i * s)];
    }
#pragma unroll
    for (int h = N >> 1; h > 0; h >>= 1) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            if ((i & h) == 0) {
                const uint64_t ah = xh[i], al = xl[i], bh = xh[i + h], bl = xl[i + h];
                const bool a_less = ah < bh || (ah == bh && al < bl);
                const bool swap = a_less == down;
                xh[i] = swap ? bh : ah;
                xl[i] = swap ? bl : al;
                xh[i + h] = swap ? ah : bh;
                xl[i + h] = swap ? al : bl;
            }
        }
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
        hi[pad(base + i * s)] = xh[i];
        lo[pad(base + i * s)] = xl[i];
    }
}

// The sort keys of the union's P entries per subgraph (old S_spec first, then the k best of S_x, then padding), one
// thread per entry: hi = score key << 32 | upper half of ~hash, lo = lower half of ~hash << 32 | ~position.  The
// schedules of the k best sit at random places of the population: many workgroups share those reads.
// (One wavefront per workgroup: the reads are random single elements of a population far larger than the caches, and
// what bounds them is how many misses a compute unit keeps in flight; the launch therefore spreads over all units.)
constexpr int kKeysThreads = 64;
__global__ void __launch_bounds__(kKeysThreads) lse_keys_kernel(const LseSeg* __restrict__ segs, int k, int P, const uint16_t* __restrict__ tiles,
                                                       int64_t pitch, const int32_t* __restrict__ best_idx, const float* __restrict__ best_val,
                                                       const uint16_t* __restrict__ old_tiles, const float* __restrict__ old_score,
                                                       const int32_t* __restrict__ old_count, int64_t spec_pitch,
                                                       uint64_t* __restrict__ key_hi, uint64_t* __restrict__ key_lo)
{
    const int s = blockIdx.y;
    const int i = blockIdx.x * kKeysThreads + threadIdx.x;
    if (i >= P) return;
    const int n_slots = segs[s].n_slots;
    const int64_t col0 = (int64_t)s * k;
    const int n_old = old_count[s] < 0 ? 0 : old_count[s] > k ? k : old_count[s];
    uint64_t h = 0, l = 0;   // padding sorts last: every real entry has a non-zero key
    if (i < n_old + k) {
        float sc;
        uint64_t hash;
        if (i < n_old) {
            sc = old_score[col0 + i];
            hash = schedule_hash(old_tiles + col0 + i, spec_pitch, n_slots);
        } else {
            const int r = i - n_old;
            sc = best_val[col0 + r];
            hash = schedule_hash(tiles + best_idx[col0 + r], pitch, n_slots);
        }
        const uint64_t inv = ~hash;
        h = ((uint64_t)lse_key_of(sc) << 32) | (inv >> 32);
        l = (inv << 32) | (uint64_t)(0xFFFFFFFFu - (uint32_t)i);
    }
    key_hi[(int64_t)s * P + i] = h;
    key_lo[(int64_t)s * P + i] = l;
}

// One workgroup per subgraph.  The old S_spec arrives in order (it is an earlier call's output: keys strictly
// descending), so only the k best of S_x are sorted (Pn = 2^m >= k entries, padding last), and the union's order is
// a merge: an entry's place is its place in its own list plus the number of entries of the other list that precede
// it, found by bisection.  Dynamic LDS: the old keys (2 x k words), the new ones (2 x padded(Pn) words), and which
// entry holds each place of the union (2 k half-words).  P is the stride of the key arrays.
__device__ __forceinline__ bool key_greater(uint64_t ah, uint64_t al, uint64_t bh, uint64_t bl) { return ah > bh || (ah == bh && al > bl); }

__global__ void __launch_bounds__(kLseThreads) lse_merge_kernel(int k, int P, int Pn, const uint64_t* __restrict__ key_hi,
                                                                const uint64_t* __restrict__ key_lo, const int32_t* __restrict__ best_idx,
                                                                const int32_t* __restrict__ old_count, float* __restrict__ new_score,
                                                                int32_t* __restrict__ new_count, int32_t* __restrict__ source)
{
    extern __shared__ uint64_t words[];
    uint64_t* oh = words;
    uint64_t* ol = oh + k;
    uint64_t* hi = ol + k;
    uint64_t* lo = hi + padded(Pn);
    uint16_t* who = reinterpret_cast<uint16_t*>(lo + padded(Pn));
    __shared__ uint32_t wave_tot[kLseThreads / kWave];
    const int s = blockIdx.x;
    const int64_t col0 = (int64_t)s * k;
    const int n_old = old_count[s] < 0 ? 0 : old_count[s] > k ? k : old_count[s];
    const int m = n_old + k;
    for (int i = threadIdx.x; i < n_old; i += kLseThreads) {
        oh[i] = key_hi[(int64_t)s * P + i];
        ol[i] = key_lo[(int64_t)s * P + i];
    }
    for (int i = threadIdx.x; i < Pn; i += kLseThreads) {
        hi[pad(i)] = i < k ? key_hi[(int64_t)s * P + n_old + i] : 0ull;   // padding sorts last: every real entry has a non-zero key
        lo[pad(i)] = i < k ? key_lo[(int64_t)s * P + n_old + i] : 0ull;
    }
    // bitonic sort, largest (hi, lo) first; one round trip through LDS performs up to three consecutive strides
    // (a thread takes the 8, 4 or 2 entries those strides permute among themselves and exchanges them in registers)
    for (int size = 2; size <= Pn; size <<= 1) {
        int stride = size >> 1;
        while (stride > 0) {
            __syncthreads();
            if (stride >= 4) {
                const int st = stride >> 2;
                for (int g = threadIdx.x; g < (Pn >> 3); g += kLseThreads) sort_group<3>(hi, lo, g, st, size);
                stride >>= 3;
            } else if (stride == 2) {
                for (int g = threadIdx.x; g < (Pn >> 2); g += kLseThreads) sort_group<2>(hi, lo, g, 1, size);
                stride = 0;
            } else {
                for (int g = threadIdx.x; g < (Pn >> 1); g += kLseThreads) sort_group<1>(hi, lo, g, 1, size);
                stride = 0;
            }
        }
    }
    __syncthreads();
    // places in the union (all 128-bit keys differ: they carry the position)
    for (int i = threadIdx.x; i < m; i += kLseThreads) {
        const bool is_old = i < n_old;
        const int j = is_old ? i : i - n_old;
        const uint64_t xh = is_old ? oh[j] : hi[pad(j)], xl = is_old ? ol[j] : lo[pad(j)];
        int a = 0, e = is_old ? k : n_old;   // entries of the other list that are greater
        while (a < e) {
            const int mid = (a + e) >> 1;
            const bool g = is_old ? key_greater(hi[pad(mid)], lo[pad(mid)], xh, xl) : key_greater(oh[mid], ol[mid], xh, xl);
            if (g) a = mid + 1; else e = mid;
        }
        who[j + a] = (uint16_t)(is_old ? j : k + j);
    }
    __syncthreads();
    // a copy has the key and the hash of its predecessor; number the rest.  A thread takes kPer neighbouring places, so
    // that one scan over the workgroup numbers a whole sweep of kPer * kLseThreads places (all 2 k of them as a rule).
    constexpr int kPer = 8;
    uint32_t carry = 0;
    for (int base = 0; base < m; base += kPer * kLseThreads) {
        const int first = base + (int)threadIdx.x * kPer;
        uint64_t mh[kPer], ml[kPer];
        uint32_t keep = 0;   // bit j: place first + j stays
        uint64_t ph = 0, pl = 0;
        if (first > 0 && first < m) {
            const int pid = who[first - 1];
            ph = pid < k ? oh[pid] : hi[pad(pid - k)];
            pl = pid < k ? ol[pid] : lo[pad(pid - k)];
        }
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            mh[j] = ml[j] = 0;
            if (first + j < m) {
                const int id = who[first + j];
                mh[j] = id < k ? oh[id] : hi[pad(id - k)];
                ml[j] = id < k ? ol[id] : lo[pad(id - k)];
                const bool same = first + j > 0 && mh[j] == ph && (ml[j] >> 32) == (pl >> 32);
                keep |= same ? 0u : 1u << j;
                ph = mh[j], pl = ml[j];
            }
        }
        // exclusive scan of the kept counts over the workgroup
        const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
        const uint32_t mine = (uint32_t)__popc(keep);
        const uint32_t incl = wave_inclusive_sum(mine);
        __syncthreads();
        if (lane == kWave - 1) wave_tot[wave] = incl;
        __syncthreads();
        uint32_t before = 0, all = 0;
        for (int w2 = 0; w2 < kLseThreads / kWave; ++w2) {
            const uint32_t t = wave_tot[w2];
            before += w2 < wave ? t : 0u;
            all += t;
        }
        uint32_t rank = carry + before + incl - mine;
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            if ((keep >> j) & 1u) {
                if (rank < (uint32_t)k) {
                    const uint32_t pos = 0xFFFFFFFFu - (uint32_t)ml[j];
                    new_score[col0 + rank] = lse_score_of((uint32_t)(mh[j] >> 32));
                    source[col0 + rank] = pos < (uint32_t)n_old ? -1 - (int32_t)pos : best_idx[col0 + (pos - n_old)];
                }
                ++rank;
            }
        }
        carry += all;
    }
    const uint32_t count = carry < (uint32_t)k ? carry : (uint32_t)k;
    for (int r = count + threadIdx.x; r < k; r += kLseThreads) {
        new_score[col0 + r] = -__builtin_inff();
        source[col0 + r] = kNoSource;
    }
    if (threadIdx.x == 0) new_count[s] = (int32_t)count;
}

// ---- short segments: selection and PriorFilter in one launch -----------------------------------------------------------
// One workgroup of 1024 threads per subgraph; thread t holds entries t, t + 1024, ... of the segment as keys.
//   1. the key of rank k: histograms of 2048 bins over the range the keys span, then over the range of the bin that holds
//      rank k, and so on until that bin holds exactly what is still to take, or few entries (then ranked by counting), or one
//      key value only (then its first entries in index order are taken).  Keys are ordered like logarithms: a bin of the
//      first pass is a fraction of a per cent to a few per cent of a score;
//   2. the chosen entries' schedules (one per thread; from the second step on the draft kernels leave the children as records
//      too, a record being one or two requests where a column's rows are one each), their hashes, and their order by (score,
//      hash, age): every wavefront sorts its 64 in registers, and neighbouring runs are merged, an entry's place being its
//      place in its run plus, by bisection, the greater ones in the other;
//   3. the union with the old S_spec, whose keys come in order from the step before, as in lse_merge; every thread then
//      writes the record it holds to the record's new place.
// Bound: the latency of these dependent stages (a compute unit works alone on a subgraph).  8,000 entries, k = 512: 23 us
// where selection (26), keys (9), merge (18) and copy (7) took 60 in four launches.

constexpr int kShortPer = 32;
constexpr int kShortMax = kLseThreads * kShortPer;   // entries of a segment
constexpr int kShortK = 1024;                        // S_spec: one old and one new member per thread
constexpr int kShortBin = 256;                       // entries of rank k's bin that are ranked by counting instead of split further

__device__ __forceinline__ void wave_sort_descending(uint64_t& hi, uint64_t& lo)   // the wavefront's 64 pairs over its lanes, largest first
{
    const int lane = lane_id();
    auto exchange = [&](auto stride_c, int size) {
        constexpr int stride = decltype(stride_c)::value;
        const uint64_t oh = lane_xor_u64<stride>(hi), ol = lane_xor_u64<stride>(lo);
        const bool lower = (lane & stride) == 0, down = (lane & size) == 0;
        const bool keep = (lower == down) == key_greater(hi, lo, oh, ol);
        hi = keep ? hi : oh;
        lo = keep ? lo : ol;
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
}

// S_spec between the steps of the short route: its keys in order and its records, by subgraph
struct ShortSpec {
    uint64_t *hi, *lo;   // [n_sg][k]
    uint4* aos;          // [n_sg][k][kAosSlots / 8]
    int32_t* count;      // [n_sg]
};

// PER: entries of a segment per thread (the longest segment decides).  first: there is no S_spec yet.  spec_tiles,
// spec_score and spec_count are written when they are not null (the last step).
template <int PER>
__global__ void __launch_bounds__(kLseThreads) lse_select_kernel(const LseSeg* __restrict__ segs, int k, bool first, const float* __restrict__ score,
                                                                 const uint16_t* __restrict__ tiles, int64_t pitch,
                                                                 const uint4* __restrict__ child_aos /* or null */, ShortSpec before, ShortSpec now,
                                                                 int64_t spec_pitch, int rows, uint16_t* __restrict__ spec_tiles,
                                                                 float* __restrict__ spec_score, int32_t* __restrict__ spec_count)
{
    __shared__ uint32_t hist[kBins];                 // later: which entry holds each place of the union, and its rank in the new S_spec
    __shared__ __attribute__((aligned(16))) uint64_t list_hi[2 * kShortK], list_lo[2 * kShortK];   // the chosen entries: sorted runs, merged from one half into the other (list_hi
                                                                       // first holds the chosen words, list_lo the words of rank k's bin)
    __shared__ uint64_t old_hi[kShortK], old_lo[kShortK];
    __shared__ __attribute__((aligned(16))) uint16_t record[kShortK * kAosSlots];   // the chosen entries' schedules
    __shared__ uint32_t wave_tot[16], found[3], low_of[16], high_of[16];
    __shared__ uint32_t fill, bin_fill, bin_rank[kShortBin];
    uint16_t* who = reinterpret_cast<uint16_t*>(hist);
    uint16_t* rank_of = who + 2 * kShortK;
    static_assert(sizeof(hist) >= 4 * kShortK * sizeof(uint16_t), "places and ranks of the union's 2 k entries");
    const int s = blockIdx.x, tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const LseSeg seg = segs[s];
    const int len = (int)(seg.end - seg.begin);
    const int64_t col0 = (int64_t)s * k;

    uint32_t key[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int i = j * kLseThreads + tid;
        key[j] = i < len ? key_of(score[seg.begin + i]) : 0u;   // 0 is below every key of a number
    }
    // Thread t holds the chosen entry t and, for an S_spec of at most half the threads, old member t - kLseThreads / 2 (the two
    // groups then work side by side), else old member t.
    const bool side_by_side = k <= kLseThreads / 2;
    const int old_at = side_by_side ? tid - kLseThreads / 2 : tid;
    // the old S_spec travels meanwhile
    int n_old = first ? 0 : before.count[s];
    n_old = n_old < 0 ? 0 : n_old > k ? k : n_old;
    uint64_t oh = 0, ol = 0;
    uint4 old_rec[kAosSlots / 8];
    const bool has_old = old_at >= 0 && old_at < n_old;
    if (has_old) {
        oh = before.hi[col0 + old_at];
        ol = before.lo[col0 + old_at];
#pragma unroll
        for (int q = 0; q < kAosSlots / 8; ++q) old_rec[q] = before.aos[(col0 + old_at) * (kAosSlots / 8) + q];
    }

    // 1. the key of rank k
    {
        uint32_t hi_key = 0, inv_lo = 0;   // the largest key, and the largest complement of one
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            hi_key = key[j] > hi_key ? key[j] : hi_key;
            const uint32_t inv = key[j] ? ~key[j] : 0u;
            inv_lo = inv > inv_lo ? inv : inv_lo;
        }
        hi_key = wave_inclusive_max(hi_key);
        inv_lo = wave_inclusive_max(inv_lo);
        if (lane == kWave - 1) {
            high_of[wave] = hi_key;
            low_of[wave] = inv_lo;
        }
        if (tid == 0) fill = bin_fill = 0;
        if (tid < kShortBin) bin_rank[tid] = 0;
    }
    __syncthreads();
    uint32_t lo_key, width;   // the keys lo_key .. lo_key + width hold rank k
    {
        uint32_t h = 0, l = 0;
#pragma unroll
        for (int w = 0; w < kLseThreads / kWave; ++w) {
            h = high_of[w] > h ? high_of[w] : h;
            l = low_of[w] > l ? low_of[w] : l;
        }
        lo_key = ~l;
        width = h - lo_key;
    }
    uint32_t k_rem = (uint32_t)k, in_bin;
    for (;;) {
        const int bits = width ? 32 - __clz(width) : 0, shift = bits > 11 ? bits - 11 : 0;
        for (int i = tid; i < kBins; i += kLseThreads) hist[i] = 0;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            if (j * kLseThreads < len) light_hist_add(hist, (key[j] - lo_key) >> shift, key[j] != 0u && key[j] - lo_key <= width);
        }
        __syncthreads();
        find_bucket(hist, k_rem, wave_tot, found);
        lo_key += found[0] << shift;
        width = (1u << shift) - 1u;
        k_rem = found[1];
        in_bin = found[2];
        __syncthreads();
        if (shift == 0 || in_bin == k_rem || in_bin <= (uint32_t)kShortBin) break;
    }
    // entries above the bin are taken; of the bin's all, or the best k_rem: by rank among a few, or (ties) in index order
    const bool all = in_bin == k_rem, few = !all && in_bin <= (uint32_t)kShortBin, ties = !all && !few;
    if (ties) {
        // ties of each (round j, wavefront), numbered in index order: one scan over PER x 16 counts
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const unsigned long long m = __ballot(key[j] == lo_key);
            if (lane == 0) hist[j * 16 + wave] = (uint32_t)__popcll(m);
        }
        __syncthreads();
        uint32_t total;
        const uint32_t c = tid < PER * 16 ? hist[tid] : 0u;
        const uint32_t before_mine = block_excl_scan<kLseThreads>(c, wave_tot, &total);
        if (tid < PER * 16) hist[tid] = before_mine;
        __syncthreads();
    }
    {
        uint32_t take = 0, in_few = 0;   // bit j: entry j is chosen / goes to the list of the bin's few
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const bool in = key[j] != 0u && key[j] - lo_key <= width;
            bool chosen = key[j] > lo_key && (!in || all);
            chosen = chosen || (in && all);
            if (ties) {
                const unsigned long long m = __ballot(in);
                chosen = chosen || (in && hist[j * 16 + wave] + (uint32_t)__popcll(m & ((1ull << lane) - 1ull)) < k_rem);
            }
            take |= chosen ? 1u << j : 0u;
            in_few |= in && few ? 1u << j : 0u;
        }
        // (both counts of a thread in one word: a workgroup holds at most 2^15 entries)
        const uint32_t mine = (uint32_t)__popc(take) | ((uint32_t)__popc(in_few) << 16);
        const uint32_t upto = wave_inclusive_sum(mine);
        uint32_t base = 0, few_base = 0;
        if (lane == kWave - 1) {
            if (upto & 0xFFFFu) base = atomicAdd(&fill, upto & 0xFFFFu);
            if (upto >> 16) few_base = atomicAdd(&bin_fill, upto >> 16);
        }
        uint32_t at = (uint32_t)__builtin_amdgcn_readlane((int)base, kWave - 1) + ((upto - mine) & 0xFFFFu);
        uint32_t at_few = (uint32_t)__builtin_amdgcn_readlane((int)few_base, kWave - 1) + ((upto - mine) >> 16);
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const uint32_t i = (uint32_t)(j * kLseThreads + tid);
            if ((take >> j) & 1u) {
                if (at < (uint32_t)k) list_hi[at] = compose(key[j], i);
                ++at;
            }
            if ((in_few >> j) & 1u) {
                if (at_few < (uint32_t)kShortBin) list_lo[at_few] = compose(key[j], i);
                ++at_few;
            }
        }
    }
    __syncthreads();
    if (few) {
        const int n_bin = (int)in_bin, e = tid & (kShortBin - 1), quarter = tid / kShortBin;
        static_assert(kLseThreads == 4 * kShortBin, "four threads count for an entry");
        const uint64_t me = e < n_bin ? list_lo[e] : ~0ull;
        uint32_t greater = 0;
        const int per = (n_bin + 3) >> 2, from = quarter * per, to = from + per < n_bin ? from + per : n_bin;
#pragma unroll 4
        for (int x = from; x < to; ++x) greater += list_lo[x] > me ? 1u : 0u;
        if (e < n_bin && greater) atomicAdd(&bin_rank[e], greater);
        __syncthreads();
        if (tid < n_bin && bin_rank[tid] < k_rem) {
            const uint32_t at = atomicAdd(&fill, 1u);
            if (at < (uint32_t)k) list_hi[at] = me;
        }
        __syncthreads();
    }

    // 2. the chosen entries' schedules, one per thread.  (The loops from here on are kept rolled: a workgroup runs this code
    // once, and most of what unrolled code would cost is its way into the instruction cache.)
    uint64_t nh = 0, nl = 0;
    const bool has_new = tid < k;
    if (has_new) {
        const uint64_t w = list_hi[tid];
        const uint32_t i = index_of(w) < (uint32_t)len ? index_of(w) : 0u;   // (always inside the segment)
        uint16_t* rec = record + tid * kAosSlots;
        if (child_aos) {
            const uint4* from = child_aos + (seg.begin + i) * (kAosSlots / 8);
            uint4 p[kAosSlots / 8];
#pragma unroll
            for (int q = 0; q < kAosSlots / 8; ++q) {
                p[q] = make_uint4(0u, 0u, 0u, 0u);
                if (8 * q < seg.n_slots) p[q] = from[q];
            }
#pragma unroll
            for (int q = 0; q < kAosSlots / 8; ++q) *reinterpret_cast<uint4*>(rec + 8 * q) = p[q];
        } else {
            const uint16_t* col = tiles + seg.begin + i;
            uint16_t f[kAosSlots];
#pragma unroll
            for (int r = 0; r < kAosSlots; ++r) f[r] = r < PRUNER_MAX_SLOTS && r < seg.n_slots ? col[r * pitch] : (uint16_t)0;
#pragma unroll
            for (int q = 0; q < kAosSlots / 8; ++q) {
                uint32_t p[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) p[e] = (uint32_t)f[8 * q + 2 * e] | ((uint32_t)f[8 * q + 2 * e + 1] << 16);
                *reinterpret_cast<uint4*>(rec + 8 * q) = make_uint4(p[0], p[1], p[2], p[3]);
            }
        }
        uint64_t h = (uint64_t)seg.n_slots;
#pragma unroll 1
        for (int r = 0; r < seg.n_slots; ++r) h = splitmix64_draw(h, (uint64_t)rec[r] + 1);
        const uint64_t inv = ~h;
        nh = (w & 0xFFFFFFFF00000000ull) | (inv >> 32);
        nl = (inv << 32) | (uint64_t)(0xFFFFFFFFu - ((uint32_t)k + i));   // younger than S_spec's members, then by index
    }
    if (has_old) {
        old_hi[old_at] = oh;
        old_lo[old_at] = ol;
    }
    int sorted = kWave;   // 64 or the power of two at or above k
    while (sorted < k) sorted <<= 1;
    if (!has_new) nl = (uint64_t)tid;   // fillers: behind every entry (no entry has hi = 0), and distinct
    __syncthreads();   // the chosen words have been read
    if (tid < sorted) {
        uint64_t sh = nh, sl = nl;
        wave_sort_descending(sh, sl);
        list_hi[tid] = sh;
        list_lo[tid] = sl;
    }
    __syncthreads();
    // entries of a run of n that are greater than (xh, xl)
    auto greater_in = [](const uint64_t* hi, const uint64_t* lo, int n, uint64_t xh, uint64_t xl) {
        int a = 0;
#pragma unroll 1
        for (int step = 1 << (31 - __clz(n | 1)); step > 0; step >>= 1) {
            const bool there = a + step <= n;
            const int at = there ? a + step - 1 : 0;
            a += there && key_greater(hi[at], lo[at], xh, xl) ? step : 0;
        }
        return a;
    };
    int rank = 0, from = 0;   // the entry's place in its run; the half of the lists that holds the runs
    if (tid < sorted) rank = greater_in(list_hi + 64 * wave, list_lo + 64 * wave, kWave, nh, nl);
#pragma unroll 1
    for (int run = kWave; run < sorted; run *= 2) {
        if (tid < sorted) {
            const int other = from + ((tid & ~(run - 1)) ^ run);
            rank += greater_in(list_hi + other, list_lo + other, run, nh, nl);
            const int to = (from ^ kShortK) + (tid & ~(2 * run - 1)) + rank;
            list_hi[to] = nh;
            list_lo[to] = nl;
        }
        from ^= kShortK;
        __syncthreads();
    }
    const uint64_t *new_hi = list_hi + from, *new_lo = list_lo + from;   // all chosen entries in order

    // 3. places in the union (all 128-bit keys differ: they carry the age): one's own rank and the greater ones of the other list
    int place_new = 0, place_old = 0;
    if (side_by_side) {
        const bool mine_new = tid < kLseThreads / 2;
        const int greater = greater_in(mine_new ? old_hi : new_hi, mine_new ? old_lo : new_lo, mine_new ? n_old : k, mine_new ? nh : oh, mine_new ? nl : ol);
        place_new = rank + greater;
        place_old = old_at + greater;
    } else {
        place_new = rank + greater_in(old_hi, old_lo, n_old, nh, nl);
        place_old = old_at + greater_in(new_hi, new_lo, k, oh, ol);
    }
    if (has_new) who[place_new] = (uint16_t)(kShortK + rank);
    if (has_old) who[place_old] = (uint16_t)old_at;
    __syncthreads();
    const int m = n_old + k;
    uint32_t keep = 0;
    {
        uint64_t ph = 0, pl = 0;
#pragma unroll
        for (int j = -1; j < 2; ++j) {
            const int at = 2 * tid + j;
            uint64_t xh = 0, xl = 0;
            if (at >= 0 && at < m) {
                const int id = who[at];
                xh = id < kShortK ? old_hi[id] : new_hi[id - kShortK];
                xl = id < kShortK ? old_lo[id] : new_lo[id - kShortK];
            }
            // a copy has the key and the hash of its predecessor
            if (j >= 0 && at < m && !(at > 0 && xh == ph && (xl >> 32) == (pl >> 32))) keep |= 1u << j;
            ph = xh, pl = xl;
        }
    }
    uint32_t total;
    const uint32_t at_rank = block_excl_scan<kLseThreads>((uint32_t)__popc(keep), wave_tot, &total);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const uint32_t r = at_rank + (j == 1 ? keep & 1u : 0u);
        if (2 * tid + j < m) rank_of[2 * tid + j] = (keep >> j) & 1u && r < (uint32_t)k ? (uint16_t)r : (uint16_t)0xFFFFu;
    }
    __syncthreads();
    const uint32_t count = total < (uint32_t)k ? total : (uint32_t)k;
    auto write = [&](int r, uint64_t xh, uint64_t xl, const uint4 (&w)[kAosSlots / 8]) {
        now.hi[col0 + r] = xh;
        now.lo[col0 + r] = (xl & 0xFFFFFFFF00000000ull) | (uint64_t)(0xFFFFFFFFu - (uint32_t)r);
#pragma unroll
        for (int q = 0; q < kAosSlots / 8; ++q) now.aos[(col0 + r) * (kAosSlots / 8) + q] = w[q];
        if (spec_tiles) {
            spec_score[col0 + r] = lse_score_of((uint32_t)(xh >> 32));
#pragma unroll
            for (int q = 0; q < kAosSlots / 8; ++q) {
                const uint4 v = w[q];
                const uint32_t p[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (8 * q + e < PRUNER_MAX_SLOTS && 8 * q + e < rows) spec_tiles[(8 * q + e) * spec_pitch + col0 + r] = (uint16_t)(p[e >> 1] >> (16 * (e & 1)));
            }
        }
    };
    const int r_new = has_new ? (int)rank_of[place_new] : 0xFFFF, r_old = has_old ? (int)rank_of[place_old] : 0xFFFF;
#pragma unroll 1
    for (int turn = side_by_side ? 1 : 0; turn < 2; ++turn) {   // (side by side a thread has one of the two)
        const bool mine_new = side_by_side ? tid < kLseThreads / 2 : turn == 0;
        const int r = mine_new ? r_new : r_old;
        uint4 w[kAosSlots / 8];
#pragma unroll
        for (int q = 0; q < kAosSlots / 8; ++q) {
            const uint4 mine = *reinterpret_cast<const uint4*>(record + tid * kAosSlots + 8 * q);
            w[q] = make_uint4(mine_new ? mine.x : old_rec[q].x, mine_new ? mine.y : old_rec[q].y, mine_new ? mine.z : old_rec[q].z, mine_new ? mine.w : old_rec[q].w);
        }
        if (r != 0xFFFF) write(r, mine_new ? nh : oh, mine_new ? nl : ol, w);
    }
    if (tid == 0) now.count[s] = (int32_t)count;
    if (spec_tiles) {
        if (tid == 0) spec_count[s] = (int32_t)count;
        for (int r = (int)count + tid; r < k; r += kLseThreads) {
            spec_score[col0 + r] = -__builtin_inff();
            for (int row = 0; row < rows; ++row) spec_tiles[row * spec_pitch + col0 + r] = 0;
        }
    }
}

// The tile factors of the new S_spec; rows a subgraph does not own and entries past the count are cleared.  A second
// copy holds each schedule's factors side by side (32 x uint16 = 64 bytes): the mutation reads a parent from there
// with four loads instead of one per factor.
__global__ void __launch_bounds__(256) lse_copy_kernel(const LseSeg* __restrict__ segs, int n_sg, int k, int rows, const uint16_t* __restrict__ tiles,
                                                       int64_t pitch, const uint16_t* __restrict__ old_tiles, int64_t spec_pitch,
                                                       const int32_t* __restrict__ source, uint16_t* __restrict__ new_tiles,
                                                       uint4* __restrict__ new_aos)
{
    const int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (c >= (int64_t)n_sg * k) return;
    const int s = (int)(c / k);
    const int n_slots = segs[s].n_slots;
    const int32_t src = source[c];
    uint32_t packed[kAosSlots / 2];
#pragma unroll
    for (int i = 0; i < kAosSlots / 2; ++i) packed[i] = 0u;
#pragma unroll
    for (int row = 0; row < PRUNER_MAX_SLOTS; ++row) {
        uint16_t v = 0;
        if (row < n_slots && src != kNoSource) v = src < 0 ? old_tiles[row * spec_pitch + (int64_t)s * k + (-1 - src)] : tiles[row * pitch + src];
        if (row < rows) new_tiles[row * spec_pitch + c] = v;
        packed[row >> 1] |= (uint32_t)v << (16 * (row & 1));
    }
#pragma unroll
    for (int q = 0; q < kAosSlots / 8; ++q) new_aos[c * (kAosSlots / 8) + q] = make_uint4(packed[4 * q], packed[4 * q + 1], packed[4 * q + 2], packed[4 * q + 3]);
}

// The segment of child j: the last one that begins at or before j (empty ones are skipped over).
__device__ __forceinline__ int lse_segment_of(const LseSeg* __restrict__ segs, int n_sg, int64_t j)
{
    int lo = 0, hi = n_sg - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (segs[mid].begin <= j) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// VEC children of one subgraph, neighbours in the population, and their stores (one per row when VEC > 1)
template <int VEC, int NP>
__device__ __forceinline__ void lse_children(const LseSeg& seg, int sub, int count, int k, uint64_t z0, const uint4* __restrict__ spec_aos,
                                             uint32_t mutate_q16, uint16_t* __restrict__ tiles, int64_t pitch, int64_t j0)
{
    uint32_t f[VEC][kAosWords];
#pragma unroll
    for (int e = 0; e < VEC; ++e) lse_child<NP>(seg, sub, count, k, z0 + (uint64_t)(2 * e) * kGamma, spec_aos, mutate_q16, f[e]);
#pragma unroll
    for (int row = 0; row < 8 * NP && row < PRUNER_MAX_SLOTS; ++row) {
        if (row < seg.n_slots) {
            if constexpr (VEC == 1) {
                tiles[row * pitch + j0] = (uint16_t)(f[0][row >> 1] >> (16 * (row & 1)));
            } else {
                // the row's factor of each child: the low or the high halves of two children's words at a time
                const uint32_t half = row & 1 ? 0x07060302u : 0x05040100u;
                const uint32_t w01 = __builtin_amdgcn_perm(f[1 % VEC][row >> 1], f[0][row >> 1], half);
                if constexpr (VEC == 4) {
                    const uint32_t w23 = __builtin_amdgcn_perm(f[3 % VEC][row >> 1], f[2 % VEC][row >> 1], half);
                    *reinterpret_cast<uint2*>(tiles + row * pitch + j0) = make_uint2(w01, w23);
                } else {
                    *reinterpret_cast<uint32_t*>(tiles + row * pitch + j0) = w01;
                }
            }
        }
    }
}
template <int VEC>
__device__ __forceinline__ void lse_children(const LseSeg& seg, int sub, int count, int k, uint64_t z0, const uint4* __restrict__ spec_aos,
                                             uint32_t mutate_q16, uint16_t* __restrict__ tiles, int64_t pitch, int64_t j0)
{
    switch ((seg.n_slots + 7) >> 3) {   // (the same for a whole wavefront but at a border between subgraphs)
        case 0:
        case 1: lse_children<VEC, 1>(seg, sub, count, k, z0, spec_aos, mutate_q16, tiles, pitch, j0); break;
        case 2: lse_children<VEC, 2>(seg, sub, count, k, z0, spec_aos, mutate_q16, tiles, pitch, j0); break;
        case 3: lse_children<VEC, 3>(seg, sub, count, k, z0, spec_aos, mutate_q16, tiles, pitch, j0); break;
        default: lse_children<VEC, 4>(seg, sub, count, k, z0, spec_aos, mutate_q16, tiles, pitch, j0); break;
    }
}

// VEC children per thread (neighbours in the population), stored VEC at a time.
// VEC > 1 needs a pitch that is a multiple of VEC and a population aligned to 2 VEC bytes.
template <int VEC>
__global__ void __launch_bounds__(256) lse_mutate_kernel(const LseSeg* __restrict__ segs, int n_sg, int k, int64_t n, uint16_t* __restrict__ tiles,
                                                         int64_t pitch, const uint4* __restrict__ spec_aos,
                                                         const int32_t* __restrict__ spec_count, uint64_t seed, uint64_t step,
                                                         uint32_t mutate_q16)
{
    const int64_t j0 = ((int64_t)blockIdx.x * 256 + threadIdx.x) * VEC;
    if (j0 >= n) return;
    const int sub = lse_segment_of(segs, n_sg, j0);
    const LseSeg seg = segs[sub];
    const uint64_t z0 = lse_child_state(seed, step, j0);
    if (VEC > 1 && j0 + VEC <= seg.end) {
        // all of this thread's children belong to one subgraph: one store per row
        const int count = spec_count[sub];
        if (count < 1) return;
        lse_children<VEC>(seg, sub, count, k, z0, spec_aos, mutate_q16, tiles, pitch, j0);
        return;
    }
    // a thread at a border between subgraphs (or VEC = 1): child by child
    for (int e = 0; e < VEC; ++e) {
        const int64_t j = j0 + e;
        if (j >= n) return;
        const int sj = e == 0 ? sub : lse_segment_of(segs, n_sg, j);
        const LseSeg sg = segs[sj];
        const int count = spec_count[sj];
        if (count < 1 || j >= sg.end) continue;
        lse_children<1>(sg, sj, count, k, z0 + (uint64_t)(2 * e) * kGamma, spec_aos, mutate_q16, tiles, pitch, j);
    }
}

struct LseLayout {
    size_t filter, table, best_idx, best_val, alt_tiles, alt_score, alt_count, zero_count, source, key_hi, key_lo, aos, aos_b, children, total;
};

LseLayout lse_layout(int64_t n, int32_t n_sg, int32_t k, int32_t rows)
{
    LseLayout L;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off += round_up(bytes, 256);
        return at;
    };
    const size_t cols = (size_t)n_sg * (size_t)k;
    L.filter = take(prior_filter_workspace_bytes(n, n_sg, k));
    L.table = take((size_t)n_sg * sizeof(LseSeg));
    L.best_idx = take(cols * sizeof(int32_t));
    L.best_val = take(cols * sizeof(float));
    L.alt_tiles = take((size_t)rows * cols * sizeof(uint16_t));
    L.alt_score = take(cols * sizeof(float));
    L.alt_count = take((size_t)n_sg * sizeof(int32_t));
    L.zero_count = take((size_t)n_sg * sizeof(int32_t));
    L.source = take(cols * sizeof(int32_t));
    L.key_hi = take(4 * cols * sizeof(uint64_t));   // P < 4k entries per subgraph (2k rounded up to a power of two)
    L.key_lo = take(4 * cols * sizeof(uint64_t));
    L.aos = take(cols * kAosSlots * sizeof(uint16_t));
    // the short route's records take turns, and so a population that may take it has its children as records
    const bool may_be_short = k <= kShortK && n <= (int64_t)n_sg * kShortMax;
    L.aos_b = take((may_be_short ? cols : 0) * kAosSlots * sizeof(uint16_t));
    L.children = take((may_be_short ? (size_t)n : 0) * kAosSlots * sizeof(uint16_t));
    L.total = off;
    return L;
}

PerDeviceFlag g_merge_ready;   // the merge kernel's allowance of dynamic LDS has been raised

}  // namespace

size_t lse_workspace_bytes(int64_t n, int32_t n_sg, int32_t k, int32_t rows)
{
    if (n < 0) n = 0;
    if (n_sg < 1) n_sg = 1;
    if (k < 1) k = 1;
    if (rows < 1) rows = 1;
    return lse_layout(n, n_sg, k, rows).total;
}

}  // namespace pruner

using namespace pruner;

extern "C" int pruner_lse(const pruner_subgraph* sg, int32_t n_sg, const int64_t* seg_off, uint16_t* tiles, int64_t tiles_pitch,
                          int32_t tile_rows, int32_t flags, int32_t k, int32_t n_steps, uint64_t seed, uint32_t mutate_q16, float* score,
                          uint16_t* spec_tiles, float* spec_score, int32_t* spec_count, void* workspace, size_t workspace_bytes,
                          void* stream)
{
    if (!sg || !seg_off || n_sg < 1 || n_sg > PRUNER_MAX_SUBGRAPHS) return PRUNER_EINVAL;
    if (n_steps < 1 || mutate_q16 > 65536 || k < 1 || k > PRUNER_MAX_K || tile_rows < 1 || tile_rows > PRUNER_MAX_SLOTS) return PRUNER_EINVAL;
    if (!spec_tiles || !spec_score || !spec_count || !aligned(spec_tiles, 2) || !aligned(spec_score, 4) || !aligned(spec_count, 4))
        return PRUNER_EINVAL;
    if (!workspace || !aligned(workspace, 256)) return PRUNER_EWORKSPACE;
    const int64_t n = seg_off[n_sg];
    if (n < 0 || n > 0x7FFFFFFFll) return PRUNER_EINVAL;
    const LseLayout L = lse_layout(n, n_sg, k, tile_rows);
    if (workspace_bytes < L.total) return PRUNER_EWORKSPACE;
    char* ws = static_cast<char*>(workspace);
    hipStream_t st = static_cast<hipStream_t>(stream);

    // everything the draft and selection stages refuse, before the first launch
    const size_t draft_bytes = round_up(draft_workspace_bytes(n_sg), 256);
    int rc = draft_check(sg, n_sg, seg_off, tiles, tiles_pitch, flags, score, nullptr, ws + L.filter, draft_bytes);
    if (rc) return rc;
    std::vector<LseSeg> table(n_sg);
    for (int32_t s = 0; s < n_sg; ++s) {
        if (seg_off[s + 1] - seg_off[s] < k) return PRUNER_EINVAL;
        const int32_t n_slots = sg[s].n_sp * 4 + sg[s].n_rd * sg[s].rd_levels;
        if (n_slots > tile_rows) return PRUNER_EINVAL;
        const bool frag = sg[s].frag[0] != 0 || sg[s].frag[1] != 0 || sg[s].frag[2] != 0;
        table[s] = LseSeg{seg_off[s], seg_off[s + 1], sg[s].n_sp, sg[s].n_rd, sg[s].rd_levels, n_slots,
                          {frag ? sg[s].frag[0] : 0, frag ? sg[s].frag[1] : 0, frag ? sg[s].frag[2] : 0}, 0};
    }

    int P = 2;
    while (P < 2 * k) P <<= 1;
    int Pn = 2;
    while (Pn < k) Pn <<= 1;
    const size_t merge_lds = (size_t)k * 16 + (size_t)padded(Pn) * 16 + (size_t)k * 4;
    const int dev = current_device(nullptr);
    if (dev < 0) return PRUNER_EHIP;
    if (!g_merge_ready.get(dev)) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(&lse_merge_kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)(PRUNER_MAX_K * 20 + padded(PRUNER_MAX_K) * 16)) != hipSuccess)
            return PRUNER_EHIP;
        g_merge_ready.mark(dev);
    }

    LseSeg* d_table = reinterpret_cast<LseSeg*>(ws + L.table);
    int32_t* best_idx = reinterpret_cast<int32_t*>(ws + L.best_idx);
    float* best_val = reinterpret_cast<float*>(ws + L.best_val);
    int32_t* source = reinterpret_cast<int32_t*>(ws + L.source);
    int32_t* zero_count = reinterpret_cast<int32_t*>(ws + L.zero_count);
    uint64_t* key_hi = reinterpret_cast<uint64_t*>(ws + L.key_hi);
    uint64_t* key_lo = reinterpret_cast<uint64_t*>(ws + L.key_lo);
    uint4* aos = reinterpret_cast<uint4*>(ws + L.aos);
    // S_spec alternates between the caller's arrays and the workspace's, ending in the caller's
    uint16_t* spec_t[2] = {spec_tiles, reinterpret_cast<uint16_t*>(ws + L.alt_tiles)};
    float* spec_s[2] = {spec_score, reinterpret_cast<float*>(ws + L.alt_score)};
    int32_t* spec_n[2] = {spec_count, reinterpret_cast<int32_t*>(ws + L.alt_count)};
    const int64_t spec_pitch = (int64_t)n_sg * k;

    auto mutate = [&](int32_t t, const int32_t* count, const uint4* records) {   // SchMutation of step t, in place (parents come from S_spec, not from S_x)
        if (tiles_pitch % 4 == 0 && aligned(tiles, 8))
            hipLaunchKernelGGL(lse_mutate_kernel<4>, dim3((unsigned)((n + 1023) / 1024)), dim3(256), 0, st, d_table, n_sg, k, n, tiles, tiles_pitch,
                               records, count, seed, (uint64_t)t, mutate_q16);
        else
            hipLaunchKernelGGL(lse_mutate_kernel<1>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, d_table, n_sg, k, n, tiles, tiles_pitch,
                               records, count, seed, (uint64_t)t, mutate_q16);
    };
    void* const draft_ws = ws + L.filter;

    // The short route: every segment in one workgroup's registers, S_spec's members one per thread.
    int64_t longest = 0;
    for (int32_t s = 0; s < n_sg; ++s) longest = seg_off[s + 1] - seg_off[s] > longest ? seg_off[s + 1] - seg_off[s] : longest;
    if (longest <= kShortMax && k <= kShortK) {
        DraftPlan plan;
        rc = draft_plan(sg, n_sg, seg_off, tiles, tiles_pitch, flags, score, nullptr, draft_ws, draft_bytes, false, n_steps > 1, &plan);
        if (rc) return rc;
        // all tables in one launch: this route has no selection workspace, the segment table stands in its place
        d_table = reinterpret_cast<LseSeg*>(ws + L.filter + draft_bytes);
        Upload pending;
        pending.bytes.assign(reinterpret_cast<const char*>(table.data()), reinterpret_cast<const char*>(table.data() + table.size()));
        pending.dst = d_table;
        rc = draft_upload(plan, draft_ws, st, &pending);
        if (rc) return rc;
        uint64_t* const keys[2] = {key_hi, key_lo};
        const ShortSpec spec[2] = {ShortSpec{keys[0], keys[0] + spec_pitch, aos, zero_count},
                                   ShortSpec{keys[1], keys[1] + spec_pitch, reinterpret_cast<uint4*>(ws + L.aos_b), reinterpret_cast<int32_t*>(ws + L.alt_count)}};
        for (int32_t t = 0; t < n_steps; ++t) {
            const ShortSpec &now = spec[t & 1], &before = spec[(t & 1) ^ 1];
            uint4* const children = reinterpret_cast<uint4*>(ws + L.children);
            const MutArgs owed{d_table, before.aos, before.count, seed, (uint64_t)(t - 1), mutate_q16, k, children};
            const bool made = t > 0 && plan.makes;
            if (t > 0 && !plan.makes) {
                mutate(t - 1, before.count, before.aos);
                PRUNER_LAUNCH_CHECK();
            }
            rc = draft_run(plan, draft_ws, tiles, score, nullptr, st, nullptr, nullptr, 1, made ? &owed : nullptr);
            if (rc) return rc;
            const bool last = t + 1 == n_steps;
            uint16_t* const to_tiles = last ? spec_tiles : nullptr;
            float* const to_score = last ? spec_score : nullptr;
            int32_t* const to_count = last ? spec_count : nullptr;
#define PRUNER_SELECT(PER) hipLaunchKernelGGL(lse_select_kernel<PER>, dim3((unsigned)n_sg), dim3(kLseThreads), 0, st, d_table, k, t == 0, score, tiles, tiles_pitch, made ? children : nullptr, before, now, \
                                              spec_pitch, tile_rows, to_tiles, to_score, to_count)
            if (longest <= 8 * kLseThreads) PRUNER_SELECT(8);
            else PRUNER_SELECT(kShortPer);
#undef PRUNER_SELECT
            PRUNER_LAUNCH_CHECK();
        }
        mutate(n_steps - 1, spec_count, spec[(n_steps - 1) & 1].aos);
        PRUNER_LAUNCH_CHECK();
        return PRUNER_OK;
    }

    // the table, and the "no S_spec yet" counts of the first step, in one launch
    rc = put_table(d_table, table.data(), table.size() * sizeof(LseSeg), st, zero_count, round_up((size_t)n_sg * sizeof(int32_t), 4));
    if (rc) return rc;

    const size_t filter_bytes = L.table - L.filter;
    // The mutation of step t - 1 is owed when step t begins: the draft kernels of step t make, store and score the
    // children in one pass if their launch shape allows it, else it runs as a launch of its own first.
    DraftPlan plan_first, plan_later;
    for (int32_t t = 0; t < n_steps; ++t) {
        const int now = (n_steps - 1 - t) & 1, before = now ^ 1;   // the last step writes the caller's arrays (index 0)
        // C_SA over S_x and its k best: the launches of pruner_prior_filter
        TopkCtx ctx;
        Upload pending;
        rc = topk_prepare(seg_off, n_sg, k, ws + L.filter + draft_bytes, filter_bytes - draft_bytes, st, &ctx, &pending, true, true);
        if (rc) return rc;
        if (t == 0) rc = draft_plan(sg, n_sg, seg_off, tiles, tiles_pitch, flags, score, nullptr, draft_ws, draft_bytes, ctx.large, false, &plan_first);
        if (t == 1) rc = draft_plan(sg, n_sg, seg_off, tiles, tiles_pitch, flags, score, nullptr, draft_ws, draft_bytes, ctx.large, true, &plan_later);
        if (rc) return rc;
        const DraftPlan& plan = t == 0 ? plan_first : plan_later;
        const MutArgs owed{d_table, aos, spec_n[before], seed, (uint64_t)(t - 1), mutate_q16, k, nullptr};
        if (t > 0 && !plan.makes) {
            mutate(t - 1, spec_n[before], aos);
            PRUNER_LAUNCH_CHECK();
        }
        if (pending.dst) ctx.d_segs = place_behind(plan, draft_ws, &pending);
        rc = draft_upload(plan, draft_ws, st, &pending);
        if (rc) return rc;
        rc = draft_run(plan, draft_ws, tiles, score, nullptr, st, ctx.large ? ctx.d_hist : nullptr, ctx.large ? ctx.d_block_max : nullptr, ctx.copies,
                       t > 0 && plan.makes ? &owed : nullptr);
        if (rc) return rc;
        rc = topk_finish(ctx, score, seg_off, best_idx, best_val, ctx.large && plan.counts, st);
        if (rc) return rc;
        // PriorFilter over the union, then the new S_spec's tile factors
        const int32_t* old_n = t == 0 ? zero_count : spec_n[before];
        hipLaunchKernelGGL(lse_keys_kernel, dim3((unsigned)((P + kKeysThreads - 1) / kKeysThreads), (unsigned)n_sg), dim3(kKeysThreads), 0, st, d_table, k, P, tiles, tiles_pitch,
                           best_idx, best_val, spec_t[before], spec_s[before], old_n, spec_pitch, key_hi, key_lo);
        PRUNER_LAUNCH_CHECK();
        hipLaunchKernelGGL(lse_merge_kernel, dim3(n_sg), dim3(kLseThreads), merge_lds, st, k, P, Pn, key_hi, key_lo, best_idx, old_n, spec_s[now],
                           spec_n[now], source);
        PRUNER_LAUNCH_CHECK();
        hipLaunchKernelGGL(lse_copy_kernel, dim3((unsigned)((spec_pitch + 255) / 256)), dim3(256), 0, st, d_table, n_sg, k, tile_rows, tiles,
                           tiles_pitch, spec_t[before], spec_pitch, source, spec_t[now], aos);
        PRUNER_LAUNCH_CHECK();
    }
    // the last step's mutation: S_x as the caller receives it
    mutate(n_steps - 1, spec_n[0], aos);
    PRUNER_LAUNCH_CHECK();
    return PRUNER_OK;
}
