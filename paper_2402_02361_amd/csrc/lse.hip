// Latent Schedule Explorer (Alg. 2) with the population resident on the device:
//   n_steps times { costs = C_SA(S_x);  S_spec = PriorFilter(S_x U S_spec);  S_x = SchMutation(S_x, costs) }.
//
// C_SA and the k best of S_x are the launches of pruner_prior_filter.  The rest of a step:
//   lse_keys    sixteen lanes per schedule: the records, score keys and schedule hashes of the k best (they sit at random
//               places of the population); of children that are not stored, lse_keys_made: one lane makes a child again
//   lse_rank    every entry's place in the union of S_spec and the k best: the order is (score descending, hash ascending,
//               position ascending); S_spec is in that order already, the k best in runs, places are found by bisection
//   lse_unite   the union as a union of SETS (a schedule counts once; identity = score and a 64-bit hash of the tile
//               factors): copies of a predecessor are dropped, the first k of the rest are the new S_spec; one 64-byte record
//               per schedule, from which the mutation reads its parents
//   lse_mutate  one thread per child: a parent drawn uniformly from S_spec (truncation selection: the paper names a
//               genetic algorithm guided by the draft fitness and gives no operator), and with the given probability
//               one prime factor of one tile factor moved to another level of the same axis, fragment multiples kept
// Short segments with a small S_spec (kShortMax entries, k up to kShortK, but see spread_out: the populations of an ordinary tuning round)
// take one launch for the selection and all of PriorFilter instead:
//   lse_select  one workgroup per subgraph: the k best of S_x from keys in registers, their schedules' hashes, the union
//               with S_spec and the new S_spec's records
// When the population gets one draft launch per loop-nest class (or one for several closed forms, where all children are looked up, below), the
// mutation of a step is not a launch of its own: the next step's draft kernels make the children and score them while they are in registers.  They are not stored: a child is a
// function of the seed, the step, its number and S_spec, and the few that are chosen are made again where they are wanted; only the
// last step's mutation, whose children nobody scores, is a launch that stores them.
// Where a segment has many times more children than S_spec can have different ones (a child is one of some thirty to a few hundred moves
// away from its parent), all of these are made and scored first, and the children's scores are looked up: a child then costs its two
// draws.  21 million children of two subgraphs, k = 4096, a step: 58 + 8 us for the table, where making, storing and scoring every child took
// 221 (the call of four steps 1,334 -> 874).
// Random numbers are counter-based (SplitMix64, Steele/Lea/Flood OOPSLA 2014: draw c is the c-th output of the
// generator started from the seed), so the result does not depend on how the work is laid out.
#include "lse_child.h"
#include "select_common.h"

#include <string.h>

#include <vector>

namespace pruner {
namespace {

__device__ __forceinline__ uint64_t splitmix64_draw(uint64_t seed, uint64_t c)
{
    uint64_t z = seed + c * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__device__ __forceinline__ uint32_t lse_key_of(float x)   // larger score <=> larger key; -0 and +0 share a key
{
    uint32_t u = __float_as_uint(x);
    if (u == 0x80000000u) u = 0u;
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float lse_score_of(uint32_t key) { return __uint_as_float((key & 0x80000000u) ? (key & 0x7FFFFFFFu) : ~key); }

__device__ __forceinline__ bool key_greater(uint64_t ah, uint64_t al, uint64_t bh, uint64_t bl) { return ah > bh || (ah == bh && al > bl); }

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

// S_spec between the steps: its sort keys in order and its records, by subgraph.  A sort key is 128 bits, larger first:
// hi = score key << 32 | upper half of ~hash, lo = lower half of ~hash << 32 | ~position in the union.
struct Spec {
    uint64_t *hi, *lo;   // [n_sg][k]
    uint4* aos;          // [n_sg][k][kAosSlots / 8]
    int32_t* count;      // [n_sg]
};

__device__ __forceinline__ int spec_members(const int32_t* count, int s, int k)
{
    const int n = count[s];
    return n < 0 ? 0 : n > k ? k : n;
}

// ---- PriorFilter over the union of S_spec and the k best, for segments of any length: lse_keys, lse_rank, lse_unite ------
// Three launches over the whole device instead of a sort by one workgroup per subgraph.  21 million programs in one segment,
// k = 4096, a step: 11 + 7 + 6 us, where keys, sort and copies took 22 + 53 + 10.

// The records and sort keys of the k best of S_x, 64 per workgroup, which leaves their keys in order.
constexpr int kRun = kWave;   // neighbours of the k best whose keys are in order
struct Fresh {
    uint64_t *hi, *lo;   // [n_sg][k]
    uint32_t* aos;       // [n_sg][k][kAosWords]
};

// ... from their records in LDS, one to a lane of a wavefront
__device__ __forceinline__ void leave_keys(const uint32_t (*record)[kAosWords + 1], int s, int k, int n_slots, int n_old, const float* __restrict__ best_val, const Fresh& fresh)
{
    const int64_t col0 = (int64_t)s * k;
    const int mine = blockIdx.x * kRun + (int)threadIdx.x;
    const float score = mine < k ? best_val[col0 + mine] : 0.f;
    uint64_t hi = 0, lo = 0;   // padding sorts last: every real entry has a key above 0
    if (mine < k) {
        uint64_t h = (uint64_t)n_slots;   // identity of a schedule: its own tile slots, in slot order
        for (int row = 0; row < n_slots; ++row) {
            const uint32_t pair = record[threadIdx.x][row >> 1];
            h = splitmix64_draw(h, (uint64_t)(row & 1 ? pair >> 16 : pair & 0xFFFFu) + 1);
        }
        const uint64_t inv = ~h;
        const uint32_t position = (uint32_t)(n_old + mine);
        hi = ((uint64_t)lse_key_of(score) << 32) | (inv >> 32);
        lo = (inv << 32) | (uint64_t)(0xFFFFFFFFu - position);
    }
    wave_sort_descending(hi, lo);
    if (mine < k) {
        fresh.hi[col0 + mine] = hi;
        fresh.lo[col0 + mine] = lo;
    }
}

// Schedules of a population sit at random places, two bytes a row: sixteen lanes per schedule, so that all misses are under way at once.
__global__ void __launch_bounds__(kLseThreads) lse_keys_kernel(const LseSeg* __restrict__ segs, int k, bool first, const int32_t* __restrict__ old_count,
                                                               const uint16_t* __restrict__ tiles, int64_t pitch, const int32_t* __restrict__ best_idx,
                                                               const float* __restrict__ best_val, Fresh fresh)
{
    static_assert(kLseThreads == kRun * kAosWords, "a thread takes two slots of a schedule");
    __shared__ uint32_t record[kRun][kAosWords + 1];
    const int s = blockIdx.y, c = threadIdx.x / kAosWords, w = threadIdx.x % kAosWords;
    const int n_slots = segs[s].n_slots;
    const int64_t col0 = (int64_t)s * k;
    const int r = blockIdx.x * kRun + c;
    uint32_t word = 0;
    if (r < k) {
        const uint16_t* col = tiles + best_idx[col0 + r];
        const uint32_t low = 2 * w < n_slots ? col[(int64_t)(2 * w) * pitch] : 0u, high = 2 * w + 1 < n_slots ? col[(int64_t)(2 * w + 1) * pitch] : 0u;
        word = low | high << 16;
        fresh.aos[(col0 + r) * kAosWords + w] = word;
    }
    record[c][w] = word;
    __syncthreads();
    if (threadIdx.x < kRun) leave_keys(record, s, k, n_slots, first ? 0 : spec_members(old_count, s, k), best_val, fresh);
}

// Children that the draft kernels made are not stored and are made again here, one by a lane.  A workgroup is one wavefront: the chain of a
// child's draws, its parent and its prime factors is long, and what hides it are other wavefronts (1,000 subgraphs, k = 1,025, four steps:
// extents with primes above 40,000 2,794 us by one wavefront of sixteen, 2,011 so; powers of two 2,018 and 1,760).
__global__ void __launch_bounds__(kRun) lse_keys_made_kernel(int k, MutArgs made, const int32_t* __restrict__ best_idx, const float* __restrict__ best_val, Fresh fresh)
{
    __shared__ uint32_t record[kRun][kAosWords + 1];
    const int s = blockIdx.y, first = blockIdx.x * kRun, child = first + (int)threadIdx.x;
    const LseSeg seg = made.segs[s];
    const int count = made.spec_count[s];
    const int64_t col0 = (int64_t)s * k;
    if (child < k) {
        uint32_t packed[kAosWords];
        lse_child<kAosSlots / 8>(seg, s, count, k, lse_child_state(made.seed, made.step, best_idx[col0 + child]), made.spec_aos, made.mutate_q16, packed);
#pragma unroll
        for (int i = 0; i < kAosWords; ++i) record[threadIdx.x][i] = packed[i];
    }
    __syncthreads();
    const int words = (k - first < kRun ? k - first : kRun) * kAosWords;
#pragma unroll
    for (int j = 0; j < kAosWords; ++j) {
        const int i = j * kRun + (int)threadIdx.x;
        if (i < words) fresh.aos[(col0 + first) * kAosWords + i] = record[i / kAosWords][i % kAosWords];
    }
    leave_keys(record, s, k, seg.n_slots, count < 0 ? 0 : count > k ? k : count, best_val, fresh);
}

// How many of the SIZE (a power of two) keys in descending order at hi, lo are above each of xh, xl.
template <int SIZE> __device__ __forceinline__ uint32_t count_above(const uint64_t* hi, const uint64_t* lo, uint64_t xh, uint64_t xl)
{
    uint32_t n = 0;
#pragma unroll
    for (int step = SIZE / 2; step > 0; step >>= 1) n += key_greater(hi[n + step - 1], lo[n + step - 1], xh, xl) ? (uint32_t)step : 0u;
    return n + (key_greater(hi[n], lo[n], xh, xl) ? 1u : 0u);
}

// Every entry's place in the union's order: 64 entries of one list per workgroup, one to a lane of each wavefront.  S_spec is
// in that order already, the k best are in runs of 64: a place is the number of greater entries in each run and, for one of the
// k best, in S_spec, found by bisection, the runs and the windows of S_spec shared out over the wavefronts.  (Comparing with
// every entry of the same score instead took 12 us without shared scores, 41 us with the many that later steps have.)
// Dynamic LDS: both lists' keys.
constexpr int kOldWindow = 256;
__host__ __device__ constexpr int rank_words(int k) { return (k + kRun - 1) / kRun * kRun + (k + kOldWindow - 1) / kOldWindow * kOldWindow; }
__global__ void __launch_bounds__(kLseThreads) lse_rank_kernel(int k, bool first, int groups, Spec before, const uint64_t* __restrict__ fresh_hi,
                                                               const uint64_t* __restrict__ fresh_lo, uint64_t* __restrict__ union_hi,
                                                               uint64_t* __restrict__ union_lo)
{
    constexpr int kWaves = kLseThreads / kWave, kRuns = PRUNER_MAX_K / kRun / kWaves;   // runs per wavefront, at most
    static_assert(PRUNER_MAX_K <= kWaves * kOldWindow, "a window of S_spec per wavefront");
    extern __shared__ uint64_t words[];
    __shared__ uint32_t place[kWave];
    const int s = blockIdx.y, lane = lane_id(), wave = threadIdx.x >> 6, runs = (k + kRun - 1) / kRun;
    const int64_t col0 = (int64_t)s * k;
    const int n_old = first ? 0 : spec_members(before.count, s, k);
    // this workgroup's groups of 64 entries: those of S_spec are counted first, then those of the k best
    const int g0 = (int)blockIdx.x * groups, g1 = g0 + groups < 2 * runs ? g0 + groups : 2 * runs;
    if (g1 <= runs && g0 * kRun >= n_old) return;
    const int n_fresh = runs * kRun, n_window = g1 <= runs ? 0 : (n_old + kOldWindow - 1) / kOldWindow * kOldWindow;
    uint64_t *hi = words, *lo = hi + n_fresh, *oh = lo + n_fresh, *ol = oh + n_window;
    for (int i = threadIdx.x; i < n_fresh; i += kLseThreads) {
        hi[i] = i < k ? fresh_hi[col0 + i] : 0ull;
        lo[i] = i < k ? fresh_lo[col0 + i] : 0ull;
    }
    for (int i = threadIdx.x; i < n_window; i += kLseThreads) {
        oh[i] = i < n_old ? before.hi[col0 + i] : 0ull;
        ol[i] = i < n_old ? before.lo[col0 + i] : 0ull;
    }
#pragma unroll 1
    for (int g = g0; g < g1; ++g) {
        const bool old_side = g < runs;
        const int base = (g - (old_side ? 0 : runs)) * kRun;
        const int left = (old_side ? n_old : k) - base, n_mine = left < kRun ? left : kRun;
        if (n_mine <= 0) continue;
        uint64_t my_hi = ~0ull, my_lo = ~0ull;
        if (lane < n_mine) {
            my_hi = (old_side ? before.hi : fresh_hi)[col0 + base + lane];
            my_lo = (old_side ? before.lo : fresh_lo)[col0 + base + lane];
        }
        if (threadIdx.x < kWave) place[threadIdx.x] = old_side ? base + threadIdx.x : 0;
        __syncthreads();
        uint32_t above = 0;
#pragma unroll
        for (int j = 0; j < kRuns; ++j) {
            const int run = j * kWaves + wave;
            if (run < runs) above += count_above<kRun>(hi + run * kRun, lo + run * kRun, my_hi, my_lo);
        }
        if (!old_side && wave * kOldWindow < n_window) above += count_above<kOldWindow>(oh + wave * kOldWindow, ol + wave * kOldWindow, my_hi, my_lo);
        if (above) atomicAdd(&place[lane], above);
        __syncthreads();
        if ((int)threadIdx.x < n_mine) {
            const uint32_t at = place[lane];
            if (at < 2u * (uint32_t)k) {   // (all keys differ: they hold the position)
                union_hi[2 * col0 + at] = my_hi;
                union_lo[2 * col0 + at] = my_lo;
            }
        }
        __syncthreads();   // (the places are written again)
    }
}

// The union as a set, 64 PER places per workgroup: an entry with the score and the hash of its predecessor is a copy; the others'
// ranks are the number of such entries before them (every workgroup counts those before its own places itself: 128 KB at
// most, against a launch more).  The first k are the new S_spec; the last step writes the caller's arrays as well.
// PER = 4 where there are workgroups for several rounds of the device: fewer of them count what lies before theirs (200
// subgraphs, k = 1025: 39 -> 16 us).
template <int PER> __global__ void __launch_bounds__(kLseThreads) lse_unite_kernel(int k, bool first, Spec before, const uint32_t* __restrict__ fresh_aos,
                                                                const uint64_t* __restrict__ union_hi, const uint64_t* __restrict__ union_lo, Spec now,
                                                                int64_t spec_pitch, int rows, uint16_t* __restrict__ spec_tiles /* or null */,
                                                                float* __restrict__ spec_score, int32_t* __restrict__ spec_count)
{
    constexpr int kPer = 2 * PRUNER_MAX_K / kLseThreads;
    static_assert(kLseThreads == kWave * kAosWords, "a thread copies one word");
    constexpr int kPlaces = kWave * PER;
    __shared__ uint32_t before_mine, wave_kept[PER], from[kPlaces], to[kPlaces];
    const int s = blockIdx.y, lane = lane_id(), wave = threadIdx.x >> 6, base = (int)blockIdx.x * kPlaces;
    const int64_t col0 = (int64_t)s * k;
    const int n_old = first ? 0 : spec_members(before.count, s, k), m = n_old + k;
    if (base >= m) return;
    const uint64_t *uh = union_hi + 2 * col0, *ul = union_lo + 2 * col0;
    uint64_t h[kPer], ph[kPer];
    uint32_t l[kPer], pl[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int p = j * kLseThreads + (int)threadIdx.x;
        h[j] = ph[j] = 0;
        l[j] = pl[j] = 0;
        if (p < base) {
            const int q = p > 0 ? p - 1 : 0;
            h[j] = uh[p];
            l[j] = (uint32_t)(ul[p] >> 32);
            ph[j] = uh[q];
            pl[j] = (uint32_t)(ul[q] >> 32);
        }
    }
    if (threadIdx.x == 0) before_mine = 0;
    __syncthreads();
    uint32_t kept = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int p = j * kLseThreads + (int)threadIdx.x;
        kept += (uint32_t)__popcll(__ballot(p < base && (p == 0 || h[j] != ph[j] || l[j] != pl[j])));
    }
    if (lane == 0 && kept) atomicAdd(&before_mine, kept);
    __syncthreads();
    const uint32_t rank0 = before_mine;
    const bool last_places = base + kPlaces >= m;
    if (rank0 >= (uint32_t)k && !last_places) return;
    const int p = base + (int)threadIdx.x;
    uint64_t mh = 0, ml = 0;
    bool keep = false;
    if (threadIdx.x < kPlaces && p < m) {
        mh = uh[p];
        ml = ul[p];
        keep = p == 0 || mh != uh[p - 1] || (ml >> 32) != (ul[p - 1] >> 32);
    }
    const unsigned long long kept_lanes = __ballot(keep);
    if (wave < PER && lane == 0) wave_kept[wave] = (uint32_t)__popcll(kept_lanes);
    __syncthreads();
    uint32_t all_mine = 0, kept_before = 0;   // of this workgroup's places; of those before this wavefront's
#pragma unroll
    for (int w = 0; w < PER; ++w) {
        kept_before += w < wave ? wave_kept[w] : 0u;
        all_mine += wave_kept[w];
    }
    if (threadIdx.x < kPlaces) {
        const uint32_t rank = rank0 + kept_before + (uint32_t)__popcll(kept_lanes & ((1ull << lane) - 1ull));
        const bool stays = keep && rank < (uint32_t)k;
        to[threadIdx.x] = stays ? rank : 0xFFFFFFFFu;
        from[threadIdx.x] = 0xFFFFFFFFu - (uint32_t)ml;
        if (stays) {
            now.hi[col0 + rank] = mh;
            now.lo[col0 + rank] = (ml & 0xFFFFFFFF00000000ull) | (uint64_t)(0xFFFFFFFFu - rank);
            if (spec_tiles) spec_score[col0 + rank] = lse_score_of((uint32_t)(mh >> 32));
        }
    }
    __syncthreads();
    const int w = threadIdx.x % kAosWords;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int e = q * kWave + (int)threadIdx.x / kAosWords;
        if (to[e] == 0xFFFFFFFFu) continue;
        const int pos = (int)from[e];
        const uint32_t word = pos < n_old ? reinterpret_cast<const uint32_t*>(before.aos)[(col0 + pos) * kAosWords + w] : fresh_aos[(col0 + (pos - n_old)) * kAosWords + w];
        const int64_t at = col0 + to[e];
        reinterpret_cast<uint32_t*>(now.aos)[at * kAosWords + w] = word;
        if (spec_tiles) {
            if (2 * w < rows) spec_tiles[(int64_t)(2 * w) * spec_pitch + at] = (uint16_t)word;
            if (2 * w + 1 < rows) spec_tiles[(int64_t)(2 * w + 1) * spec_pitch + at] = (uint16_t)(word >> 16);
        }
    }
    if (last_places) {
        const uint32_t total = rank0 + all_mine, count = total < (uint32_t)k ? total : (uint32_t)k;
        if (threadIdx.x == 0) now.count[s] = (int32_t)count;
        if (spec_tiles) {
            if (threadIdx.x == 0) spec_count[s] = (int32_t)count;
            for (int r = (int)count + (int)threadIdx.x; r < k; r += kLseThreads) {
                spec_score[col0 + r] = -__builtin_inff();
                for (int row = 0; row < rows; ++row) spec_tiles[(int64_t)row * spec_pitch + col0 + r] = 0;
            }
        }
    }
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
//   3. the union with the old S_spec, whose keys come in order from the step before, every place found by bisection; every thread then
//      writes the record it holds to the record's new place.
// Bound: the latency of these dependent stages (a compute unit works alone on a subgraph).  8,000 entries, k = 512: 22 us
// (loads 2.5, the range of the keys 1.3, histograms 3.4, taking 2.5, records 1.5, hashes 1, sorting 1.5 and merging 2.8, the union 3.6)
// where selection (26), keys (9), merge (18) and copy (7) took 60 in four launches.

struct alignas(16) Sorted { uint64_t hi, lo; };   // a sort key

constexpr int kShortPer = 32;
constexpr int kShortMax = kLseThreads * kShortPer;   // entries of a segment
constexpr int kShortK = 1024;                        // S_spec: one old and one new member per thread
constexpr int kShortBin = 256;                       // entries of rank k's bin that are ranked by counting instead of split further

// PER: entries of a segment per thread (the longest segment decides).  first: there is no S_spec yet.  spec_tiles,
// spec_score and spec_count are written when they are not null (the last step).
template <int PER>
__global__ void __launch_bounds__(kLseThreads) lse_select_kernel(const LseSeg* __restrict__ segs, int k, bool first, const float* __restrict__ score,
                                                                 const uint16_t* __restrict__ tiles, int64_t pitch,
                                                                 const uint4* __restrict__ child_aos /* or null */, Spec before, Spec now,
                                                                 int64_t spec_pitch, int rows, uint16_t* __restrict__ spec_tiles,
                                                                 float* __restrict__ spec_score, int32_t* __restrict__ spec_count)
{
    __shared__ uint32_t hist[kBins];                 // later: which entry holds each place of the union, and its rank in the new S_spec
    __shared__ Sorted list[2 * kShortK];             // the chosen entries: sorted runs, merged from one half into the other (first: the chosen entries' places
                                                     // in the segment, in the other half the words of rank k's bin)
    __shared__ Sorted old_list[kShortK];
    __shared__ __attribute__((aligned(16))) uint16_t record[kShortK * kAosSlots];   // the chosen entries' schedules
    __shared__ uint32_t wave_tot[16], found[3], low_of[16], high_of[16];
    __shared__ uint32_t fill, bin_fill, bin_rank[kShortBin];
    uint32_t* const chosen_at = reinterpret_cast<uint32_t*>(list);
    uint64_t* const bin_word = reinterpret_cast<uint64_t*>(list + kShortK);
    uint16_t* who = reinterpret_cast<uint16_t*>(hist);
    uint16_t* rank_of = who + 2 * kShortK;
    static_assert(sizeof(hist) >= 4 * kShortK * sizeof(uint16_t), "places and ranks of the union's 2 k entries");
    const int s = blockIdx.x, tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    int n_old = first ? 0 : before.count[s];   // (asked for at once with the segment)
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
        if (shift == 0 || in_bin == k_rem || in_bin <= (uint32_t)kShortBin) break;
        // the keys that the bin holds: one value is as much as another pass would find, and shared scores are what fills bins
        uint32_t most = 0, not_least = 0;
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const bool in = key[j] != 0u && key[j] - lo_key <= width;
            most = in && key[j] > most ? key[j] : most;
            not_least = in && ~key[j] > not_least ? ~key[j] : not_least;
        }
        most = wave_inclusive_max(most);
        not_least = wave_inclusive_max(not_least);
        if (lane == kWave - 1) {
            high_of[wave] = most;
            low_of[wave] = not_least;
        }
        __syncthreads();
        most = not_least = 0;
#pragma unroll
        for (int w = 0; w < kLseThreads / kWave; ++w) {
            most = high_of[w] > most ? high_of[w] : most;
            not_least = low_of[w] > not_least ? low_of[w] : not_least;
        }
        lo_key = ~not_least;
        width = most - lo_key;
        if (width == 0u) break;
    }
    __syncthreads();
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
        // (places only: stores of keys out of the registers, each under a condition, are longer code)
#pragma unroll 1
        for (; take; take &= take - 1u, ++at)
            if (at < (uint32_t)k) chosen_at[at] = (uint32_t)((__ffs((int)take) - 1) * kLseThreads + tid);
#pragma unroll 1
        for (; in_few; in_few &= in_few - 1u, ++at_few) {
            const uint32_t i = (uint32_t)((__ffs((int)in_few) - 1) * kLseThreads + tid);
            if (at_few < (uint32_t)kShortBin) bin_word[at_few] = compose(key_of(score[seg.begin + i]), i);
        }
    }
    __syncthreads();
    if (few) {
        const int n_bin = (int)in_bin, e = tid & (kShortBin - 1), quarter = tid / kShortBin;
        static_assert(kLseThreads == 4 * kShortBin, "four threads count for an entry");
        const uint64_t me = e < n_bin ? bin_word[e] : ~0ull;
        uint32_t greater = 0;
        const int per = (n_bin + 3) >> 2, from = quarter * per, to = from + per < n_bin ? from + per : n_bin;
#pragma unroll 4
        for (int x = from; x < to; ++x) greater += bin_word[x] > me ? 1u : 0u;
        if (e < n_bin && greater) atomicAdd(&bin_rank[e], greater);
        __syncthreads();
        if (tid < n_bin && bin_rank[tid] < k_rem) {
            const uint32_t at = atomicAdd(&fill, 1u);
            if (at < (uint32_t)k) chosen_at[at] = index_of(me);
        }
        __syncthreads();
    }

    // 2. the chosen entries' schedules, one per thread.  (The loops from here on are kept rolled: a workgroup runs this code
    // once, and most of what unrolled code would cost is its way into the instruction cache.)
    uint64_t nh = 0, nl = 0;
    const bool has_new = tid < k;
    if (has_new) {
        const uint32_t i = chosen_at[tid] < (uint32_t)len ? chosen_at[tid] : 0u;   // (always inside the segment)
        const float its_score = score[seg.begin + i];
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
        nh = ((uint64_t)key_of(its_score) << 32) | (inv >> 32);
        // younger than S_spec's members, then by index; and which thread holds the record
        static_assert(((uint64_t)(kShortK + kShortMax) << 10) < (1ull << 32) && kLseThreads <= 1024, "an age and a thread in 32 bits");
        nl = (inv << 32) | (uint64_t)(0xFFFFFFFFu - ((((uint32_t)k + i) << 10) | (uint32_t)tid));
    }
    if (has_old) old_list[old_at] = Sorted{oh, ol};
    int sorted = kWave;   // 64 or the power of two at or above k
    while (sorted < k) sorted <<= 1;
    if (!has_new) nl = (uint64_t)tid;   // fillers: behind every entry (no entry has hi = 0), and distinct
    __syncthreads();   // the chosen places have been read
    // From here on thread t has the entry that the sort of its wavefront brings it.
    if (tid < sorted) {
        wave_sort_descending(nh, nl);
        list[tid] = Sorted{nh, nl};
    }
    __syncthreads();
    // entries of a run of n that are greater than (xh, xl): the run in quarters, three looks at a time
    auto greater_in = [](const Sorted* run, int n, uint64_t xh, uint64_t xl) {
        int a = 0, size = n > 1 ? 1 << (32 - __clz(n - 1)) : 1;   // a power of two at or above n
#pragma unroll 1
        for (; size >= 4; size >>= 2) {
            const int q = size >> 2;
            Sorted at[3];
            int past = 0;
#pragma unroll
            for (int i = 0; i < 3; ++i) at[i] = run[a + (i + 1) * q - 1 < n ? a + (i + 1) * q - 1 : 0];
#pragma unroll
            for (int i = 0; i < 3; ++i) past += a + (i + 1) * q <= n && key_greater(at[i].hi, at[i].lo, xh, xl) ? 1 : 0;
            a += past * q;
        }
        if (size == 2) a += a < n && key_greater(run[a].hi, run[a].lo, xh, xl) ? 1 : 0;
        if (a < n && key_greater(run[a].hi, run[a].lo, xh, xl)) ++a;
        return a;
    };
    int rank = lane, from = 0;   // the entry's place in its run; the half of the lists that holds the runs
#pragma unroll 1
    for (int run = kWave; run < sorted; run *= 2) {
        if (tid < sorted) {
            rank += greater_in(list + from + ((tid & ~(run - 1)) ^ run), run, nh, nl);
            list[(from ^ kShortK) + (tid & ~(2 * run - 1)) + rank] = Sorted{nh, nl};
        }
        from ^= kShortK;
        __syncthreads();
    }
    const Sorted* new_list = list + from;   // all chosen entries in order
    const bool is_new = nh != 0ull;         // (not a filler)
    const int holder = (int)((0xFFFFFFFFu - (uint32_t)nl) & 1023u);   // of the entry's record

    // 3. places in the union (all 128-bit keys differ: they carry the age): one's own rank and the greater ones of the other list
    int place_new = 0, place_old = 0;
    if (side_by_side) {
        const bool mine_new = tid < kLseThreads / 2;
        const int greater = greater_in(mine_new ? old_list : new_list, mine_new ? n_old : k, mine_new ? nh : oh, mine_new ? nl : ol);
        place_new = rank + greater;
        place_old = old_at + greater;
    } else {
        place_new = rank + greater_in(old_list, n_old, nh, nl);
        place_old = old_at + greater_in(new_list, k, oh, ol);
    }
    if (is_new) who[place_new] = (uint16_t)(kShortK + rank);
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
                const Sorted x = id < kShortK ? old_list[id] : new_list[id - kShortK];
                xh = x.hi;
                xl = x.lo;
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
    const int r_new = is_new ? (int)rank_of[place_new] : 0xFFFF, r_old = has_old ? (int)rank_of[place_old] : 0xFFFF;
#pragma unroll 1
    for (int turn = side_by_side ? 1 : 0; turn < 2; ++turn) {   // (side by side a thread has one of the two)
        const bool mine_new = side_by_side ? tid < kLseThreads / 2 : turn == 0;
        const int r = mine_new ? r_new : r_old;
        uint4 w[kAosSlots / 8];
#pragma unroll
        for (int q = 0; q < kAosSlots / 8; ++q) {
            const uint4 mine = *reinterpret_cast<const uint4*>(record + holder * kAosSlots + 8 * q);
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
                    // (not through the caches: a population of 0.8 GB displaces the scores and what S_spec is read from; 141.6 -> 138.9 us)
                    __builtin_nontemporal_store((uint64_t)w01 | ((uint64_t)w23 << 32), reinterpret_cast<uint64_t*>(tiles + row * pitch + j0));
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
    size_t filter, table, best_idx, best_val, zero_count, alt_count, keys[2], fresh, fresh_aos, merged, aos, aos_b, children, total;
};

// parts: with room for the lists of the selection's blocks route
LseLayout lse_layout(int64_t n, int32_t n_sg, int32_t k, int32_t rows, bool parts)
{
    LseLayout L;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off += round_up(bytes, 256);
        return at;
    };
    const size_t cols = (size_t)n_sg * (size_t)k;
    L.filter = take(prior_filter_workspace_bytes(n, n_sg, k, parts));
    L.table = take((size_t)n_sg * sizeof(LseSeg));
    L.best_idx = take(cols * sizeof(int32_t));
    L.best_val = take(cols * sizeof(float));
    L.zero_count = take((size_t)n_sg * sizeof(int32_t));
    L.alt_count = take((size_t)n_sg * sizeof(int32_t));
    for (size_t& keys : L.keys) keys = take(2 * cols * sizeof(uint64_t));   // S_spec's, in turns
    L.fresh = take(2 * cols * sizeof(uint64_t));                            // those of the k best
    L.merged = take(4 * cols * sizeof(uint64_t));                           // the union's
    L.fresh_aos = take(cols * kAosSlots * sizeof(uint16_t));
    L.aos = take(cols * kAosSlots * sizeof(uint16_t));
    L.aos_b = take(cols * kAosSlots * sizeof(uint16_t));   // S_spec's records, in turns
    // The short route has its children as records.  The room is there whatever the route: a workspace for more candidates or a
    // larger k serves every smaller call.
    const int64_t most_short = (int64_t)n_sg * kShortMax;
    L.children = take((size_t)(n < most_short ? n : most_short) * kAosSlots * sizeof(uint16_t));
    L.total = off;
    return L;
}

constexpr int64_t kSpreadChildren = 1 << 17;   // children up to which a launch makes one per thread (8,000: 6.3 -> 4.0 us)
constexpr int kMostGroups = 8;        // of 64 entries per workgroup of the rank kernel
constexpr int kManyUniters = 2048;   // workgroups of 64 places: four times what the device holds at once

PerDeviceFlag g_rank_ready;   // the rank kernel's allowance of dynamic LDS has been raised

}  // namespace

size_t lse_workspace_bytes(int64_t n, int32_t n_sg, int32_t k, int32_t rows)
{
    if (n < 0) n = 0;
    if (n_sg < 1) n_sg = 1;
    if (k < 1) k = 1;
    if (rows < 1) rows = 1;
    return lse_layout(n, n_sg, k, rows, true).total;
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
    LseLayout L = lse_layout(n, n_sg, k, tile_rows, true);
    if (workspace_bytes < L.total) L = lse_layout(n, n_sg, k, tile_rows, false);   // (the selection then takes another route)
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

    LseSeg* d_table = reinterpret_cast<LseSeg*>(ws + L.table);
    int32_t* best_idx = reinterpret_cast<int32_t*>(ws + L.best_idx);
    float* best_val = reinterpret_cast<float*>(ws + L.best_val);
    const int64_t spec_pitch = (int64_t)n_sg * k;
    auto words = [&](size_t at) { return reinterpret_cast<uint64_t*>(ws + at); };
    // S_spec alternates between two sets of arrays; the last step writes the caller's as well
    const Spec spec[2] = {Spec{words(L.keys[0]), words(L.keys[0]) + spec_pitch, reinterpret_cast<uint4*>(ws + L.aos), reinterpret_cast<int32_t*>(ws + L.zero_count)},
                          Spec{words(L.keys[1]), words(L.keys[1]) + spec_pitch, reinterpret_cast<uint4*>(ws + L.aos_b), reinterpret_cast<int32_t*>(ws + L.alt_count)}};

    auto mutate = [&](int32_t t, const int32_t* count, const uint4* records) {   // SchMutation of step t, in place (parents come from S_spec, not from S_x)
        if (n > kSpreadChildren && tiles_pitch % 4 == 0 && aligned(tiles, 8))   // (few: one to a thread, on four times the compute units)
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
    if (longest <= kShortMax && k <= kShortK && !spread_out(n, longest, n_sg, k)) {
        DraftPlan plan;
        rc = draft_plan(sg, n_sg, seg_off, tiles, tiles_pitch, flags, score, nullptr, draft_ws, draft_bytes, ScoreNotes{}, n_steps > 1 ? Makes::kChildren : Makes::kNothing, &plan);
        if (rc) return rc;
        // all tables in one launch: this route has no selection workspace, the segment table stands in its place
        d_table = reinterpret_cast<LseSeg*>(ws + L.filter + draft_bytes);
        Upload pending;
        pending.bytes.assign(reinterpret_cast<const char*>(table.data()), reinterpret_cast<const char*>(table.data() + table.size()));
        pending.dst = d_table;
        rc = draft_upload(plan, draft_ws, st, &pending);
        if (rc) return rc;
        for (int32_t t = 0; t < n_steps; ++t) {
            const Spec &now = spec[t & 1], &before = spec[(t & 1) ^ 1];
            uint4* const children = reinterpret_cast<uint4*>(ws + L.children);
            const MutArgs owed{d_table, before.aos, before.count, seed, (uint64_t)(t - 1), mutate_q16, k, children, nullptr, nullptr, 0};
            const bool made = t > 0 && plan.makes;
            if (t > 0 && !plan.makes) {
                mutate(t - 1, before.count, before.aos);
                PRUNER_LAUNCH_CHECK();
            }
            rc = draft_run(plan, draft_ws, tiles, score, nullptr, st, ScoreNotes{}, made ? &owed : nullptr);
            if (rc) return rc;
            const bool last = t + 1 == n_steps;
            uint16_t* const to_tiles = last ? spec_tiles : nullptr;
            float* const to_score = last ? spec_score : nullptr;
            int32_t* const to_count = last ? spec_count : nullptr;
#define PRUNER_SELECT(PER) hipLaunchKernelGGL(lse_select_kernel<PER>, dim3((unsigned)n_sg), dim3(kLseThreads), 0, st, d_table, k, t == 0, score, tiles, tiles_pitch, made ? children : nullptr, before, now, \
                                              spec_pitch, tile_rows, to_tiles, to_score, to_count)
            // (keys that are not there cost their places in the unrolled loops: a GEMM's 16,384, four steps, k = 64: 160 -> 132 us with 16)
            if (longest <= 8 * kLseThreads) PRUNER_SELECT(8);
            else if (longest <= 16 * kLseThreads) PRUNER_SELECT(16);
            else PRUNER_SELECT(kShortPer);
#undef PRUNER_SELECT
            PRUNER_LAUNCH_CHECK();
        }
        mutate(n_steps - 1, spec_count, spec[(n_steps - 1) & 1].aos);
        PRUNER_LAUNCH_CHECK();
        return PRUNER_OK;
    }

    const int dev = current_device(nullptr);
    if (dev < 0) return PRUNER_EHIP;
    if (!g_rank_ready.get(dev)) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(&lse_rank_kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                rank_words(PRUNER_MAX_K) * 16) != hipSuccess)
            return PRUNER_EHIP;
        g_rank_ready.mark(dev);
    }
    // Segments with many times more children than S_spec can have different ones get a table of all of these and their scores.  It
    // stands where the short route has its children as records.
    std::vector<int64_t> variant_off(n_sg + 1, 0);
    bool all_tabled = false;
    int32_t* const odd = reinterpret_cast<int32_t*>(ws + L.children);
    float* const scores_of_all = reinterpret_cast<float*>(ws + L.children + round_up((size_t)n_sg * sizeof(int32_t), 256));
    {
        const int64_t room = (int64_t)(L.total - L.children) - (int64_t)round_up((size_t)n_sg * sizeof(int32_t), 256);
        int64_t end = 0;
        int32_t n_tabled = 0;
        std::vector<int64_t> entries(n_sg, 0);
        std::vector<int> draws(n_sg, 0);
        for (int32_t s = 0; s < n_sg && n_steps > 1; ++s) entries[s] = table_entries(sg[s], seg_off[s + 1] - seg_off[s], k, &draws[s]);
        drop_partial(seg_off, n_sg, entries.data());
        for (int32_t s = 0; s < n_sg; ++s) {
            variant_off[s] = end;
            if (entries[s] == 0 || (end + entries[s]) * (int64_t)sizeof(float) > room) continue;
            table[s].table = table_word((uint32_t)end, draws[s]);
            end += entries[s];
            ++n_tabled;
        }
        variant_off[n_sg] = end;
        all_tabled = n_tabled == n_sg;
    }
    const int64_t table_end = variant_off[n_sg];
    rc = put_table(d_table, table.data(), table.size() * sizeof(LseSeg), st, table_end > 0 ? odd : nullptr, table_end > 0 ? (size_t)n_sg * sizeof(int32_t) : 0);
    if (rc) return rc;

    const size_t filter_bytes = L.table - L.filter;
    // The mutation of step t - 1 is owed when step t begins: the draft kernels of step t make and score the
    // children in one pass, or look their scores up, if their launch shape allows it, else it runs as a launch of its own first.
    DraftPlan plan_first, plan_later, plan_table;
    bool tabled = false;   // the children's scores are looked up
    for (int32_t t = 0; t < n_steps; ++t) {
        const Spec &now = spec[t & 1], &before = spec[(t & 1) ^ 1];
        // C_SA over S_x and its k best: the launches of pruner_prior_filter
        TopkCtx ctx;
        Upload pending;
        rc = topk_prepare(seg_off, n_sg, k, ws + L.filter + draft_bytes, filter_bytes - draft_bytes, st, &ctx, &pending, true, true);
        if (rc) return rc;
        const ScoreNotes notes = notes_for(ctx);
        if (t == 0) rc = draft_plan(sg, n_sg, seg_off, tiles, tiles_pitch, flags, score, nullptr, draft_ws, draft_bytes, notes, Makes::kNothing, &plan_first);
        if (rc) return rc;
        if (t == 1 && table_end > 0 && table_pays(n, plan_first.n_classes, notes.max256 || notes.first_digit)) {
            const int32_t as_they = (flags & ~(PRUNER_REFERENCE_ROUNDING | PRUNER_FUSED_ARITHMETIC)) | (plan_first.exact ? PRUNER_REFERENCE_ROUNDING : PRUNER_FUSED_ARITHMETIC);
            rc = draft_plan(sg, n_sg, variant_off.data(), tiles, table_end > tiles_pitch ? table_end : tiles_pitch, as_they, scores_of_all, nullptr, draft_ws, draft_bytes, ScoreNotes{},
                            Makes::kVariants, &plan_table);
            if (rc) return rc;
            plan_table.in_launch = true;
            tabled = fits_launch(plan_table) && plan_table.makes;
        }
        if (t == 1) {
            rc = draft_plan(sg, n_sg, seg_off, tiles, tiles_pitch, flags, score, nullptr, draft_ws, draft_bytes, notes, tabled && all_tabled ? Makes::kLookedUp : Makes::kChildren,
                            &plan_later);
            if (rc) return rc;
        }
        DraftPlan& plan = t == 0 ? plan_first : plan_later;
        const bool made = t > 0 && plan.makes;
        const MutArgs owed{d_table, before.aos, before.count, seed, (uint64_t)(t - 1), mutate_q16, k, nullptr, made && tabled ? scores_of_all : nullptr, odd, 0};
        if (t > 0 && !plan.makes) {
            mutate(t - 1, before.count, before.aos);
            PRUNER_LAUNCH_CHECK();
        }
        if (made && tabled) {
            MutArgs all = owed;
            all.table = nullptr;
            all.variants = 1;
            rc = draft_run(plan_table, draft_ws, tiles, scores_of_all, nullptr, st, ScoreNotes{}, &all);
            if (rc) return rc;
        }
        if (pending.dst) ctx.d_segs = place_behind(plan, draft_ws, &pending);
        rc = draft_upload(plan, draft_ws, st, &pending);
        if (rc) return rc;
        rc = draft_run(plan, draft_ws, tiles, score, nullptr, st, notes, made ? &owed : nullptr);
        if (rc) return rc;
        rc = topk_finish(ctx, score, seg_off, best_idx, best_val, true, st);
        if (rc) return rc;
        // PriorFilter over the union
        uint64_t* const merged = words(L.merged);
        const Fresh fresh{words(L.fresh), words(L.fresh) + spec_pitch, reinterpret_cast<uint32_t*>(ws + L.fresh_aos)};
        const dim3 runs((unsigned)((k + kRun - 1) / kRun), (unsigned)n_sg);
        if (made) hipLaunchKernelGGL(lse_keys_made_kernel, runs, dim3(kRun), 0, st, k, owed, best_idx, best_val, fresh);
        else hipLaunchKernelGGL(lse_keys_kernel, runs, dim3(kLseThreads), 0, st, d_table, k, t == 0, before.count, tiles, tiles_pitch, best_idx, best_val, fresh);
        PRUNER_LAUNCH_CHECK();
        // (a workgroup loads both lists before it ranks: where there are workgroups for several rounds of the device, which holds one
        // to two of them per compute unit, each ranks more groups.  100 subgraphs, k = 3,370, four steps: 2,269 us one group each,
        // 1,361 with eight; sixteen and thirty-two the same, 1,376 and 1,439)
        const int rank_groups = 2 * ((k + kRun - 1) / kRun);
        const int64_t rank_rounds = (int64_t)n_sg * rank_groups / 1024;
        const int groups = rank_rounds < 1 ? 1 : rank_rounds < kMostGroups ? (int)rank_rounds : kMostGroups;
        hipLaunchKernelGGL(lse_rank_kernel, dim3((unsigned)((rank_groups + groups - 1) / groups), (unsigned)n_sg), dim3(kLseThreads), (size_t)rank_words(k) * 16, st, k, t == 0,
                           groups, before, fresh.hi, fresh.lo, merged, merged + 2 * spec_pitch);
        PRUNER_LAUNCH_CHECK();
        const bool last = t + 1 == n_steps;
#define PRUNER_UNITE(PER) hipLaunchKernelGGL(lse_unite_kernel<PER>, dim3((unsigned)((2 * k + PER * kWave - 1) / (PER * kWave)), (unsigned)n_sg), dim3(kLseThreads), 0, st, k, t == 0, before, \
                                             fresh.aos, merged, merged + 2 * spec_pitch, now, spec_pitch, tile_rows, last ? spec_tiles : nullptr, last ? spec_score : nullptr, \
                                             last ? spec_count : nullptr)
        if ((int64_t)n_sg * ((2 * k + kWave - 1) / kWave) > kManyUniters) PRUNER_UNITE(4);
        else PRUNER_UNITE(1);
#undef PRUNER_UNITE
        PRUNER_LAUNCH_CHECK();
    }
    // the last step's mutation: S_x as the caller receives it
    mutate(n_steps - 1, spec[(n_steps - 1) & 1].count, spec[(n_steps - 1) & 1].aos);
    PRUNER_LAUNCH_CHECK();
    return PRUNER_OK;
}
