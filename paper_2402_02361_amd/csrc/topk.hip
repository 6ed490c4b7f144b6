// Selection of the k best entries per segment (PriorFilter of Alg. 2; the choice of S_measured in Alg. 1).
//
// Exact selection on an order-preserving 32-bit image of the scores (key): a first digit of 2048 bins, narrow where scores
// crowd (first_digit_of), and where it does not settle the matter two more digits inside its bin; ties are taken in index
// order; the k survivors are ranked by (key descending, index ascending).  Nothing depends on the order in which blocks or
// wavefronts run.
//
// Six routes, same result:
//   tiny   - segments of at most 8192 entries and k up to 64 (the final selection after the verify stage, small draft
//            populations): one launch, no digits (tiny_select in select_common.h);
//   pick   - short segments: one launch, in which several workgroups per segment hold it in registers, count the first digit, keep
//            the few entries at or above rank k's bin, and each rank their share of them (k above kLevelMostK, or without room for
//            maxima, or few blocks per selected entry: also segments of at most kPickMax entries, behind whoever counted the digit,
//            the draft kernel or a pass);
//   levels - longer ones, k up to kLevelMostK: the same launch behind whoever held the scores and left the largest key of every sixteen
//            neighbours (the draft kernel, else a pass): a workgroup holds the few blocks of sixteen that can matter;
//   blocks - a larger k of a few segments at least 768 times as long, or segments longer than kLevelMax: two launches behind whoever held the scores and left the largest key of every 256 neighbours
//            (the draft kernel, else a pass): the entries of the best blocks that reach a bound are set aside, and picked;
//   lists  - a larger k, segments of at most kListsMax: as pick, behind one more launch that goes through the spans of the segments (whole
//            16384-entry sweeps, one workgroup each) and sets the entries at or above the bin aside in a list per span; the
//            workgroups of a segment then collect from its lists (and go through the span of a list that overflowed themselves);
//   spans  - longer segments are cut into spans of whole 16384-entry sweeps, one workgroup of 1024 threads each; the scores
//            are read twice at most (first-digit histogram, which also notes the largest key of every 256 entries; then
//            everything at or above that digit's rank-k bin is set aside, a few thousand entries as a rule, and blocks of
//            256 whose largest key lies below the bin are not read again) and the later passes work on what was set aside
//            (where the bin holds too much for that, the second digit is counted first: one more reading); six launches.
#include "select_common.h"
#include "wide_load.h"

#include <string.h>

#include <vector>

namespace pruner {
namespace {

constexpr int kSmallThreads = 1024;

struct alignas(8) SegT {
    int64_t begin, end;
    int32_t first_block, pad;
};

struct alignas(16) SelState {
    uint32_t lowest;   // lowest key of the range that holds rank k (after the last pass: the key T of rank k)
    uint32_t k_rem;    // entries still to take of that range (after the last pass: ties to take)
    uint32_t n_gt;     // entries above T (after the last pass)
    uint32_t shift;    // the range's keys are split by (key - lowest) >> shift next, then by what is left
};

// ---- the selection in LDS ---------------------------------------------------------------------------------------

// The selection lives in LDS with one spare word after every 32: neighbouring threads of the sort then touch different
// banks also when they walk 8-word groups (logical index e sits in slot(e)).
constexpr int kSelWords = PRUNER_MAX_K + PRUNER_MAX_K / 32 + 2;
__device__ __forceinline__ uint32_t slot(uint32_t e) { return e + (e >> 5); }

// Bitonic sort of P = 2^m words in LDS, largest first.  One round trip through LDS performs up to three consecutive
// strides (4s, 2s, s): a thread takes the 2, 4 or 8 words base + i*s, which those strides permute among themselves,
// and exchanges them in registers.  All words of such a group lie in one half of the current merge size, so they
// share the direction.
template <int LOG> __device__ __forceinline__ void bitonic_group(uint64_t* w, int g, int s, int size)
{
    constexpr int N = 1 << LOG;
    const int base = (g / s) * (N * s) + (g % s);
    const bool down = (base & size) == 0;
    uint64_t x[N];
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = w[slot(base + i * s)];
#pragma unroll
    for (int h = N >> 1; h > 0; h >>= 1) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            if ((i & h) == 0) {
                const uint64_t a = x[i], b = x[i + h];
                const bool swap = (a < b) == down;
                x[i] = swap ? b : a;
                x[i + h] = swap ? a : b;
            }
        }
    }
#pragma unroll
    for (int i = 0; i < N; ++i) w[slot(base + i * s)] = x[i];
}

template <int NT> __device__ __forceinline__ void sort_descending(uint64_t* w, int P)
{
    for (int size = 2; size <= P; size <<= 1) {
        int stride = size >> 1;   // largest stride still to do in this merge
        while (stride > 0) {
            __syncthreads();
            if (stride >= 4) {
                const int s = stride >> 2;
                for (int g = threadIdx.x; g < (P >> 3); g += NT) bitonic_group<3>(w, g, s, size);
                stride >>= 3;
            } else if (stride == 2) {
                for (int g = threadIdx.x; g < (P >> 2); g += NT) bitonic_group<2>(w, g, 1, size);
                stride = 0;
            } else {
                for (int g = threadIdx.x; g < (P >> 1); g += NT) bitonic_group<1>(w, g, 1, size);
                stride = 0;
            }
        }
    }
    __syncthreads();
}

__host__ __device__ __forceinline__ int pow2_at_least(int k)
{
    int P = 1;
    while (P < k) P <<= 1;
    return P;
}

// Sort n selected words and write the result rows lo .. hi - 1 of one segment (hi <= n).
template <int NT>
__device__ __forceinline__ void finish_segment(uint64_t* sel, int n, int lo, int hi, const float* __restrict__ score, int32_t* __restrict__ idx_out,
                                               float* __restrict__ val_out, int64_t row, int64_t seg_begin, int64_t seg_end, int row_len)
{
    const int P = pow2_at_least(n);
    for (int i = n + threadIdx.x; i < P; i += NT) sel[slot(i)] = 0;  // below every real word
    sort_descending<NT>(sel, P);
    for (int r0 = lo + threadIdx.x; r0 < hi; r0 += 4 * NT) {
        uint32_t gi[4];
        float v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {   // the scores of four rows are requested together
            gi[u] = r0 + u * NT < hi ? index_of(sel[slot(r0 + u * NT)]) : 0xFFFFFFFFu;
            v[u] = val_out && gi[u] >= seg_begin && gi[u] < seg_end ? score[gi[u]] : 0.f;   // never read outside the segment
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (r0 + u * NT < hi) {
                idx_out[row * row_len + r0 + u * NT] = (int32_t)gi[u];
                if (val_out) val_out[row * row_len + r0 + u * NT] = v[u];
            }
        }
    }
}

// Output rows (those of the first row_len) for n of the k collected words (their positions: which[i], or first + i * stride without a list) without
// sorting: the words are distinct
// (they carry the index), so the rank of a word is the number of larger words among all k.  A wavefront holds
// R = 64, 32 or 16 of the n words at a time (the fewest lanes that still hold them all: idle lanes would cost the same
// as busy ones) and 64 / R parts of its sixteenth of the k words to compare with; the lanes of one part read the same
// word at a time (a broadcast LDS access).  Cheap when the k words' ranks are shared out over many workgroups; a full
// sort in one workgroup is better served by the bitonic network.  cnt: 128 LDS words.  All NT threads call.
template <int NT>
__device__ __forceinline__ void rank_rows(const uint64_t* sel, int k, const uint16_t* which, int first, int stride, int n, uint32_t* cnt,
                                          const float* __restrict__ score, int32_t* __restrict__ idx_out, float* __restrict__ val_out, int64_t row,
                                          int64_t seg_begin, int64_t seg_end, int row_len)
{
    typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));
    constexpr int W = NT / kWave;
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const int R = n <= 16 ? 16 : n <= 32 ? 32 : kWave, parts = kWave / R;
    const int mine_at = lane & (R - 1), piece = wave * parts + lane / R;
    // the comparison runs over the padded storage itself, two words per LDS access; the spare words and the words
    // past the last selected one hold 0 (the caller clears them), which is below every real word
    const int n_raw = ((int)slot((uint32_t)k - 1u) + 2) & ~1;
    const int per_piece = (((n_raw + W * parts - 1) / (W * parts)) + 1) & ~1;
    const int j_lo = piece * per_piece < n_raw ? piece * per_piece : n_raw, j_hi = j_lo + per_piece < n_raw ? j_lo + per_piece : n_raw;
    // (more than 64: two to a lane, so that a share a little above 64, as hashes deal them out, does not take a round more: the filter
    // of 20 x 50,000, k = 512, about 47 words a workgroup, 24.9 -> 24.2 us)
    const bool pairs = n > kWave;
    for (int e0 = 0; e0 < n; e0 += pairs ? 2 * kWave : R) {
        if (threadIdx.x < 2 * kWave) cnt[threadIdx.x] = 0;
        auto word_at = [&](int e) { return e < n ? sel[slot(which ? (uint32_t)which[e] : (uint32_t)(first + e * stride))] : ~0ull; };
        const uint64_t mine = word_at(e0 + mine_at), other = pairs ? word_at(e0 + kWave + lane) : ~0ull;
        uint32_t c = 0, d = 0;
        if (!pairs) {
#pragma unroll 4
            for (int j = j_lo; j < j_hi; j += 2) {
                const u64x2 w = *reinterpret_cast<const u64x2*>(sel + j);
                c += w.x > mine ? 1u : 0u;
                c += w.y > mine ? 1u : 0u;
            }
        } else {
#pragma unroll 4
            for (int j = j_lo; j < j_hi; j += 2) {
                const u64x2 w = *reinterpret_cast<const u64x2*>(sel + j);
                c += w.x > mine ? 1u : 0u;
                c += w.y > mine ? 1u : 0u;
                d += w.x > other ? 1u : 0u;
                d += w.y > other ? 1u : 0u;
            }
        }
        __syncthreads();
        if (c) atomicAdd(&cnt[mine_at], c);
        if (d) atomicAdd(&cnt[kWave + lane], d);
        __syncthreads();
        // (by number: a word of ones throughout is an entry, the largest key at index 0)
        if (wave == 0 ? lane < R && e0 + lane < n : pairs && wave == 1 && e0 + kWave + lane < n) {
            const uint64_t word = wave == 0 ? mine : other;
            const uint32_t r = cnt[wave * kWave + lane], gi = index_of(word);
            if (r < (uint32_t)row_len) {
                idx_out[row * row_len + r] = (int32_t)gi;
                // a key names its score (no read to wait for), except the one that -0.0 and +0.0 share
                const uint32_t key = (uint32_t)(word >> 32);
                if (val_out) val_out[row * row_len + r] = key != kZeroKey ? score_of_key(key) : gi >= seg_begin && gi < seg_end ? score[gi] : 0.f;   // never read outside the segment
            }
        }
        __syncthreads();
    }
}

// Up to kInlineSegs segment ranges travel as kernel arguments (no table upload, one launch for the whole call).
constexpr int kInlineSegs = 128;
struct InlineSegs {
    SegT s[kInlineSegs];
    __device__ __forceinline__ SegT at(int i) const { return s[i]; }
    __device__ __forceinline__ const SegT* table() const { return s; }
};
struct SegsInMemory {
    const SegT* segs;
    __device__ __forceinline__ SegT at(int i) const { return segs[i]; }
    __device__ __forceinline__ const SegT* table() const { return segs; }
};

// ---- tiny route: segments of at most 8192 entries, k at most 64 ---------------------------------------------------
// (tiny_select in select_common.h: the final selection after the verify stage and small draft populations)

template <int PER, class Table>
__global__ void __launch_bounds__(kTinyThreads) topk_tiny_kernel(const float* __restrict__ score, Table segs, int k, int32_t* __restrict__ idx_out,
                                                                 float* __restrict__ val_out)
{
    __shared__ TinyLds L;
    const SegT seg = segs.at(blockIdx.x);
    tiny_select<PER>(L, score, seg.begin, seg.end, blockIdx.x, k, idx_out, val_out);
}

// ---- spans route ------------------------------------------------------------------------------------------------
//
// Workgroups of 1024 threads each own `span` consecutive entries of one segment (span = a multiple of 16384, sized
// so that a launch is a single wave of workgroups).  No global atomics with a return value, no cross-workgroup
// order, and every launch after the first finds the digit bucket of the pass before it by itself (all workgroups
// of a segment compute the same bucket from the merged histogram; the segment's first workgroup records it):
//   hist0        LDS histogram of the first digit, merged into one of R global copies (R > 1 spreads same-address
//                atomics when few segments share many workgroups)
//   funnel       bucket of digit 0; entries above it are final and are staged as such; entries inside it are
//                candidates: staged in the workgroup's own list and counted into the second digit's histogram
//   refine       bucket of digit 1; third digit's histogram over the staged candidates
//   settle       bucket of digit 2 = the key T of rank k; candidates above T join the staged winners, candidates
//                equal to T become the staged ties
//   gather_sort  one workgroup per segment: concatenates the staged lists in workgroup (= index) order, keeps the
//                first ties, re-reads the span of a workgroup whose list overflowed, sorts, writes the result
// A workgroup whose candidate list overflows (more than kCandCap entries of its span fall into one first-digit
// bucket: scores in a very narrow band, or equal) reads its span again in refine and settle instead.

constexpr int kBigThreads = 1024;
constexpr int kBigPer = 16;
constexpr int kRow = kBigThreads * kBigPer;   // 16384 entries per sweep of a workgroup
constexpr int kStageCap = 256;                // staged winners / ties per workgroup
constexpr int kCandCap = 1024;                // staged candidates per workgroup

struct Stage {
    uint32_t n_gt, n_tie, n_cand;              // n_gt, n_tie: true counts (may exceed the capacities); n_cand: above its capacity = overflowed
    uint32_t pad;
    uint64_t gt[kStageCap];                    // composed words of entries above T, any order
    uint32_t tie[kStageCap];                   // global indices of ties, any order
    uint64_t cand[kCandCap];                   // composed words of entries in the first digit's rank-k bucket, any order
};

// One sweep of a workgroup over kRow consecutive entries starting at `row`: thread t receives kBigPer of them, four neighbours
// per 16-byte load (at any address: the memory unit asks for multiples of an element only).
// sweep_index gives the global index of the thread's j-th entry; entries at or past `hi` read as 0.
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef f32x4 f32x4_a4 __attribute__((aligned(4)));
__device__ __forceinline__ int64_t sweep_index(int64_t row, int j) { return row + ((int64_t)(j >> 2) * kBigThreads + threadIdx.x) * 4 + (j & 3); }
__device__ __forceinline__ void load_sweep(const float* __restrict__ score, int64_t row, int64_t hi, float (&val)[kBigPer])
{
#pragma unroll
    for (int q = 0; q < kBigPer / 4; ++q) {
        const int64_t i = sweep_index(row, 4 * q);
        if (i + 3 < hi) {
            const f32x4 v = *reinterpret_cast<const f32x4_a4*>(score + i);
            val[4 * q] = v.x, val[4 * q + 1] = v.y, val[4 * q + 2] = v.z, val[4 * q + 3] = v.w;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) val[4 * q + e] = i + e < hi ? score[i + e] : 0.f;
        }
    }
}

// The digit bucket that holds rank k_rem, from the merged histogram of a finished pass.  hist: kBins LDS words
// (overwritten); found: 3 LDS words (bucket, rank left inside it, its population).  All 1024 threads call.
template <int kMaxCopies>   // the most copies the pass's histogram can have (R <= kMaxCopies)
__device__ __forceinline__ void bucket_of_pass(const uint32_t* __restrict__ ghist, int R, int n_seg, int s, uint32_t k_rem,
                                               uint32_t* hist, uint32_t* wave_tot, uint32_t* found)
{
    uint32_t part[kBins / kBigThreads][kMaxCopies];   // all loads in flight together
#pragma unroll
    for (int q = 0; q < kBins / kBigThreads; ++q) {
#pragma unroll
        for (int r = 0; r < kMaxCopies; ++r)
            part[q][r] = ghist[((int64_t)(r < R ? r : 0) * n_seg + s) * kBins + q * kBigThreads + threadIdx.x];
    }
#pragma unroll
    for (int q = 0; q < kBins / kBigThreads; ++q) {
        uint32_t c = 0;
#pragma unroll
        for (int r = 0; r < kMaxCopies; ++r) c += r < R ? part[q][r] : 0u;
        hist[q * kBigThreads + threadIdx.x] = c;
    }
    __syncthreads();
    find_bucket(hist, k_rem, wave_tot, found);
}

constexpr uint32_t kCounted = 0xFFFFFFFFu;   // Stage::n_cand of a span whose entries above the second digit's bin are staged, and in n_tie the bin's counted

__global__ void __launch_bounds__(kBigThreads) hist0_kernel(const float* __restrict__ score, const SegT* __restrict__ segs, int n_seg,
                                                            int64_t span, int R, uint32_t* __restrict__ ghist /* [R][n_seg][kBins] */,
                                                            uint32_t* __restrict__ block_max /* or null */)
{
    __shared__ uint32_t hist[kBins];
    const int s = segment_of_block(segs, n_seg, blockIdx.x);
    const SegT seg = segs[s];
    for (int i = threadIdx.x; i < kBins; i += kBigThreads) hist[i] = 0;
    __syncthreads();
    const int64_t lo = seg.begin + (int64_t)(blockIdx.x - seg.first_block) * span;
    const int64_t hi = lo + span < seg.end ? lo + span : seg.end;
    for (int64_t row = lo; row < hi; row += kRow) {
        float val[kBigPer];
        load_sweep(score, row, hi, val);
        uint32_t top[kBigPer / 4] = {};
#pragma unroll
        for (int j = 0; j < kBigPer; ++j) {
            const int64_t i = sweep_index(row, j);
            const uint32_t key = key_of(val[j]);
            light_hist_add<true>(hist, first_digit_of(key), i < hi);
            if (i < hi && key > top[j >> 2]) top[j >> 2] = key;
        }
        // a wavefront's q-th load is one block of 256 neighbouring entries (spans are whole sweeps from the segment's begin)
        if (block_max) {
#pragma unroll
            for (int q = 0; q < kBigPer / 4; ++q) {
                const uint32_t m = wave_inclusive_max(top[q]);
                const int64_t first = sweep_index(row, 4 * q) - 4 * lane_id();
                if (lane_id() == 63 && first < hi) block_max[block_max_slot(first, s)] = m;
            }
        }
    }
    __syncthreads();
    flush_hist<kBigThreads>(hist, ghist, R, n_seg, s);
}

// BLK: block_max holds the largest key of every block of 256 neighbouring entries; a block whose maximum
// lies below the bucket is not read.  Wavefront w takes blocks w, w + 16, ... of the span, 64 of them per look at the
// maxima (one per lane), and reads those that are left four at a time.
// (held to 64 registers: a compute unit then holds two of these workgroups, and a launch of up to 512 runs in one round)
template <bool BLK>
__global__ void __launch_bounds__(kBigThreads) __attribute__((amdgpu_waves_per_eu(8))) funnel_kernel(const float* __restrict__ score, const SegT* __restrict__ segs, int n_seg,
                                                             int64_t span, int R, int k, const uint32_t* __restrict__ ghist0,
                                                             uint32_t* __restrict__ ghist1, SelState* __restrict__ state,
                                                             Stage* __restrict__ stage, const uint32_t* __restrict__ block_max)
{
    __shared__ uint32_t hist[kBins];
    __shared__ uint32_t wave_tot[16];
    __shared__ uint32_t found[3];
    __shared__ uint32_t n_gt, n_cand, live_blocks;
    const int s = segment_of_block(segs, n_seg, blockIdx.x);
    const SegT seg = segs[s];
    const int64_t lo = seg.begin + (int64_t)(blockIdx.x - seg.first_block) * span;
    const int64_t hi = lo + span < seg.end ? lo + span : seg.end;
    float val[kBigPer];
    const int wave = threadIdx.x >> 6;
    if (BLK && threadIdx.x == 0) live_blocks = 0;   // (the bucket search below has barriers before anyone adds to it)
    const int64_t n_blk = (hi - lo + 255) >> 8;
    uint32_t top = 0;
    // the first sweep (the first maxima) travel while the bucket is looked up
    if constexpr (BLK) {
        const int64_t b = wave + 16 * lane_id();
        if (b < n_blk) top = block_max[block_max_slot(lo + (b << 8), s)];
    } else {
        load_sweep(score, lo, hi, val);
    }
    bucket_of_pass<8>(ghist0, R, n_seg, s, (uint32_t)k, hist, wave_tot, found);
    const uint32_t k_rem = found[1];
    // A bin that the segment's lists would not hold (a population of copies): nothing is staged in this launch, which only counts
    // the second digit; the next one stages what that digit leaves.
    const bool crowded = found[2] > (uint32_t)((seg.end - seg.begin + span - 1) / span) * (uint32_t)(kCandCap / 2);
    uint32_t lowest, width;
    first_digit_range(found[0], lowest, width);
    const int shift = next_shift(width);
    if constexpr (BLK) {
        // how many of the span's (first 1024) blocks will have to be read
        const unsigned long long first_left = __ballot(top >= lowest && wave + 16 * lane_id() < n_blk);
        if (lane_id() == 0) atomicAdd(&live_blocks, (uint32_t)__popcll(first_left));
    }
    __syncthreads();
    if (blockIdx.x == seg.first_block && threadIdx.x == 0) state[s] = SelState{lowest, k_rem, (uint32_t)k - k_rem, (uint32_t)shift};
    for (int i = threadIdx.x; i < kBins; i += kBigThreads) hist[i] = 0;
    if (threadIdx.x == 0) {
        n_gt = 0;
        n_cand = crowded ? (uint32_t)kCandCap + 1u : 0u;   // (above the capacity: the list is closed)
    }
    __syncthreads();
    // Where most blocks hold an entry of the bucket (a population of copies: ties by the hundred thousand), stepping over
    // the others gains nothing and the plain sweeps, whole rows of loads in flight, are the faster way through the span.
    const bool dense = BLK && 2 * (int64_t)live_blocks > (n_blk < 16 * kWave ? n_blk : 16 * kWave);
    Stage& mine = stage[blockIdx.x];
    // The smallest score of the bin.  Nearly every entry lies below it, and one comparison tells: a wavefront steps over an
    // entry unless one of its lanes is not below (a NaN never is; the exact test follows).
    const uint32_t low_key = lowest;
    const float t0 = score_of_key(low_key);
    // What happens to one entry (every lane of the wavefront calls it, `mine_to_look_at` says whether the lane holds one).
    auto look_at = [&](float x, int64_t i, bool mine_to_look_at, bool list_open) {
        const bool there = mine_to_look_at && i < hi;
        const uint32_t key = key_of(x);
        const bool inside = there && key - lowest <= width;
        if (there && key > lowest && !inside) {
            const uint32_t at = atomicAdd(&n_gt, 1u);
            if (at < kStageCap) mine.gt[at] = compose(key, (uint32_t)i);
        } else if (inside && list_open) {
            const uint32_t at = atomicAdd(&n_cand, 1u);
            if (at < kCandCap) mine.cand[at] = compose(key, (uint32_t)i);
        }
        light_hist_add(hist, (key - lowest) >> shift, inside);
    };
    if constexpr (BLK) {
        for (int64_t g = 0; !dense && g < n_blk; g += 16 * kWave) {
            if (g > 0) {
                const int64_t b = g + wave + 16 * lane_id();
                top = b < n_blk ? block_max[block_max_slot(lo + (b << 8), s)] : 0u;
            }
            // (a lane past the span's last block holds 0 and is left out: no key of a number is 0, and low_key = 0 takes all)
            unsigned long long left = __ballot(top >= low_key && g + wave + 16 * lane_id() < n_blk);
            while (left) {
                int32_t at[4];   // (global indices are below 2^31)
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    at[u] = -1;
                    if (left) {
                        const int l = __ffsll(left) - 1;
                        left &= left - 1;
                        at[u] = (int32_t)(lo + ((g + wave + 16 * (int64_t)l) << 8)) + 4 * lane_id();
                    }
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int64_t i = at[u];
                    if (i >= 0 && i + 3 < hi) {
                        const f32x4 v = *reinterpret_cast<const f32x4_a4*>(score + i);
                        val[4 * u] = v.x, val[4 * u + 1] = v.y, val[4 * u + 2] = v.z, val[4 * u + 3] = v.w;
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e) val[4 * u + e] = i >= 0 && i + e < hi ? score[i + e] : 0.f;
                    }
                }
                // One comparison per entry tells whether it can matter at all (nearly none does; a NaN is never below,
                // the exact test on the key follows).  The few that can are then looked at together: every lane picks the
                // first such entry it holds and the wavefront goes through the motions once, again while a lane holds more.
                bool can[kBigPer], any = false;
#pragma unroll
                for (int j = 0; j < kBigPer; ++j) {
                    can[j] = at[j >> 2] >= 0 && !(val[j] < t0);
                    any = any || can[j];
                }
                const bool list_open = n_cand <= (uint32_t)kCandCap;
                while (__ballot(any) != 0ull) {
                    bool picked = false;
                    float x = 0.f;
                    int32_t i = 0;
                    any = false;
#pragma unroll
                    for (int j = 0; j < kBigPer; ++j) {
                        if (__ballot(can[j]) == 0ull) continue;
                        const bool take = can[j] && !picked;
                        x = take ? val[j] : x;
                        i = take ? at[j >> 2] + (j & 3) : i;
                        picked = picked || take;
                        can[j] = can[j] && !take;
                        any = any || can[j];
                    }
                    look_at(x, (int64_t)i, picked, list_open);
                }
            }
        }
    }
    for (int64_t row = lo; (!BLK || dense) && row < hi; row += kRow) {
        if (BLK || row > lo) load_sweep(score, row, hi, val);
        if (crowded) {
#pragma unroll
            for (int j = 0; j < kBigPer; ++j) {
                const int64_t i = sweep_index(row, j);
                const uint32_t key = key_of(val[j]);
                const bool inside = i < hi && key - lowest <= width, above = i < hi && key > lowest && !inside;
                if (__ballot(above) != 0ull) {
                    if (above) {
                        const uint32_t at = atomicAdd(&n_gt, 1u);
                        if (at < kStageCap) mine.gt[at] = compose(key, (uint32_t)i);
                    }
                }
                light_hist_add(hist, (key - lowest) >> shift, inside);
            }
            continue;
        }
        // once the candidate list has overflowed, the later passes read the span again: nothing more is staged in it
        // (the count only has to stay above the list's capacity)
        const bool list_open = n_cand <= (uint32_t)kCandCap;
#pragma unroll
        for (int j = 0; j < kBigPer; ++j) {
            // a wavefront steps over an entry unless one of its lanes is not below the bucket's smallest score
            if (__ballot(!(val[j] < t0)) == 0ull) continue;
            look_at(val[j], sweep_index(row, j), true, list_open);
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        mine.n_gt = n_gt;
        mine.n_cand = n_cand;
        mine.n_tie = 0;
    }
    flush_hist<kBigThreads>(hist, ghist1, 1, n_seg, s);   // few contributors as a rule: one copy
}

// (held to 64 registers, as the funnel: two workgroups per compute unit)
__global__ void __launch_bounds__(kBigThreads) __attribute__((amdgpu_waves_per_eu(8))) refine_kernel(const float* __restrict__ score, const SegT* __restrict__ segs, int n_seg,
                                                             int64_t span, const uint32_t* __restrict__ ghist1,
                                                             uint32_t* __restrict__ ghist2, SelState* __restrict__ state,
                                                             Stage* __restrict__ stage)
{
    __shared__ uint32_t hist[kBins];
    __shared__ uint32_t wave_tot[16];
    __shared__ uint32_t found[3];
    __shared__ uint32_t n_staged, n_gt;
    const int s = segment_of_block(segs, n_seg, blockIdx.x);
    const SegT seg = segs[s];
    const SelState before = state[s];
    bucket_of_pass<1>(ghist1, 1, n_seg, s, before.k_rem, hist, wave_tot, found);
    const uint32_t lowest = before.lowest + (found[0] << before.shift), width = (1u << before.shift) - 1u, k_rem = found[1];
    __syncthreads();
    for (int i = threadIdx.x; i < kBins; i += kBigThreads) hist[i] = 0;
    __syncthreads();
    Stage& mine = stage[blockIdx.x];
    const uint32_t n_cand = mine.n_cand;
    if (n_cand <= (uint32_t)kCandCap) {
        for (uint32_t base = 0; base < n_cand; base += kBigThreads) {
            const uint32_t i = base + threadIdx.x;
            const uint32_t key = i < n_cand ? (uint32_t)(mine.cand[i] >> 32) : 0u;
            light_hist_add(hist, key - lowest, i < n_cand && key - lowest <= width);
        }
    } else {
        // The list did not hold the bin's entries.  Those that the second digit leaves in play, in its bin and above it up to the
        // first bin's end, are staged now; where its bin alone is still too much (ties), only those above it, and the bin's
        // entries are counted span by span.  (Explorer loop, 21 M programs, a step full of copies: funnel, refine and settle
        // took 42 + 22 + 25 us with three readings of the scores, 35 + 28 + 5 with two.)
        const bool crowded = found[2] > (uint32_t)((seg.end - seg.begin + span - 1) / span) * (uint32_t)(kCandCap / 2);
        const uint32_t first_width = ((uint32_t)kBins << before.shift) - 1u;
        const int64_t lo = seg.begin + (int64_t)(blockIdx.x - seg.first_block) * span;
        const int64_t hi = lo + span < seg.end ? lo + span : seg.end;
        if (threadIdx.x == 0) {
            n_staged = 0;
            n_gt = mine.n_gt;
        }
        __syncthreads();
        uint32_t n_inside = 0;
        if (crowded) {
            const bool some_above = k_rem != before.k_rem;   // then key - next <= above_width tells them
            const uint32_t next = lowest + width + 1u, above_width = before.lowest + first_width - next;
            for (int64_t row = lo; row < hi; row += kRow) {
                float val[kBigPer];
                load_sweep(score, row, hi, val);
                const int left = hi - row < kRow ? (int)(hi - row) : kRow;
#pragma unroll
                for (int j = 0; j < kBigPer; ++j) {
                    const uint32_t key = key_of(val[j]);
                    light_hist_add(hist, key - lowest, (int)sweep_index(0, j) < left && key - lowest <= width);
                }
                bool any = false;
#pragma unroll
                for (int j = 0; j < kBigPer; ++j) any = any || key_of(val[j]) - next <= above_width;
                if (some_above && __ballot(any) != 0ull) {
#pragma unroll
                    for (int j = 0; j < kBigPer; ++j) {
                        const int i = (int)sweep_index(0, j);
                        if (i < left && key_of(val[j]) - next <= above_width) {
                            const uint32_t at = atomicAdd(&n_gt, 1u);
                            if (at < (uint32_t)kStageCap) mine.gt[at] = compose(key_of(val[j]), (uint32_t)row + (uint32_t)i);
                        }
                    }
                }
            }
        } else {
            for (int64_t row = lo; row < hi; row += kRow) {
                float val[kBigPer];
                load_sweep(score, row, hi, val);
                const int left = hi - row < kRow ? (int)(hi - row) : kRow;
#pragma unroll
                for (int j = 0; j < kBigPer; ++j) {
                    const int i = (int)sweep_index(0, j);
                    const uint32_t key = key_of(val[j]);
                    const bool in_play = i < left && key >= lowest && key - before.lowest <= first_width;
                    const unsigned long long these = __ballot(in_play);
                    if (these == 0ull) continue;
                    if (n_staged <= (uint32_t)kCandCap) {
                        const int leader = __ffsll(these) - 1;
                        uint32_t base = 0;
                        if (lane_id() == leader) base = atomicAdd(&n_staged, (uint32_t)__popcll(these));
                        const uint32_t at = (uint32_t)__builtin_amdgcn_readlane((int)base, leader) + (uint32_t)__popcll(these & ((1ull << lane_id()) - 1ull));
                        if (in_play && at < (uint32_t)kCandCap) mine.cand[at] = compose(key, (uint32_t)row + (uint32_t)i);
                    }
                    light_hist_add(hist, key - lowest, in_play && key - lowest <= width);
                }
            }
        }
        __syncthreads();
        if (crowded) {   // the span's entries inside the bin
            uint32_t inside = 0;
            for (int i = threadIdx.x; i < kBins; i += kBigThreads) inside += hist[i];
            block_excl_scan<kBigThreads>(inside, wave_tot, &n_inside);
        }
        if (threadIdx.x == 0) {
            mine.n_cand = crowded ? kCounted : n_staged;
            if (crowded) {
                mine.n_gt = n_gt;
                mine.n_tie = n_inside;
            }
        }
    }
    __syncthreads();
    flush_hist<kBigThreads>(hist, ghist2, 1, n_seg, s);
    // every workgroup of the segment has read the old state before this launch ends; the new one is for the next launch
    if (blockIdx.x == seg.first_block && threadIdx.x == 0) state[n_seg + s] = SelState{lowest, k_rem, found[2], before.shift};
}

__global__ void __launch_bounds__(kBigThreads) settle_kernel(const float* __restrict__ score, const SegT* __restrict__ segs, int n_seg,
                                                             int64_t span, int k, const uint32_t* __restrict__ ghist2,
                                                             SelState* __restrict__ state, Stage* __restrict__ stage)
{
    __shared__ uint32_t hist[kBins];
    __shared__ uint32_t wave_tot[16];
    __shared__ uint32_t found[3];
    __shared__ uint32_t n_gt, n_tie;
    const int s = segment_of_block(segs, n_seg, blockIdx.x);
    const SegT seg = segs[s];
    const SelState before = state[n_seg + s];
    bucket_of_pass<1>(ghist2, 1, n_seg, s, before.k_rem, hist, wave_tot, found);
    const uint32_t T = before.lowest + found[0], k_eq = found[1];
    __syncthreads();
    if (blockIdx.x == seg.first_block && threadIdx.x == 0) state[2 * n_seg + s] = SelState{T, k_eq, (uint32_t)k - k_eq, 0u};
    Stage& mine = stage[blockIdx.x];
    const uint32_t n_cand = mine.n_cand;
    const bool counted = n_cand == kCounted;
    if (counted && found[2] == before.n_gt) {
        // One value fills the second digit's bin: the span's ties are counted already.  Only spans before rank k that have few
        // of them need the list; the ranking reads the others itself.
        uint32_t earlier = 0;
        for (int b = seg.first_block + (int)threadIdx.x; b < (int)blockIdx.x; b += kBigThreads) earlier += stage[b].n_tie;
        uint32_t ties_before;
        block_excl_scan<kBigThreads>(earlier, wave_tot, &ties_before);
        if (mine.n_tie == 0u || mine.n_tie > (uint32_t)kStageCap || ties_before >= k_eq) return;
    }
    if (n_cand <= (uint32_t)kCandCap) {
        // winners staged so far keep their places; candidates above T follow them
        if (threadIdx.x == 0) {
            n_gt = mine.n_gt;
            n_tie = 0;
        }
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < n_cand; i += kBigThreads) {
            const uint64_t w = mine.cand[i];
            const uint32_t key = (uint32_t)(w >> 32);
            if (key > T) {
                const uint32_t at = atomicAdd(&n_gt, 1u);
                if (at < kStageCap) mine.gt[at] = w;
            } else if (key == T) {
                const uint32_t at = atomicAdd(&n_tie, 1u);
                if (at < kStageCap) mine.tie[at] = index_of(w);
            }
        }
    } else {
        // (counted: the entries above the second digit's bin, `last` its last key, are staged)
        const uint32_t last = counted ? before.lowest + ((1u << before.shift) - 1u) : 0xFFFFFFFFu;
        if (threadIdx.x == 0) {
            n_gt = counted ? mine.n_gt : 0u;
            n_tie = 0;
        }
        __syncthreads();
        const int64_t lo = seg.begin + (int64_t)(blockIdx.x - seg.first_block) * span;
        const int64_t hi = lo + span < seg.end ? lo + span : seg.end;
        for (int64_t row = lo; row < hi; row += kRow) {
            float val[kBigPer];
            load_sweep(score, row, hi, val);
#pragma unroll
            for (int j = 0; j < kBigPer; ++j) {
                const int64_t i = sweep_index(row, j);
                const uint32_t key = key_of(val[j]);
                const bool is_above = i < hi && key > T && key <= last, is_tie = i < hi && key == T;
                const unsigned long long above = __ballot(is_above), ties = __ballot(is_tie);
                if (above) {
                    if (is_above) {
                        const uint32_t at = atomicAdd(&n_gt, 1u);
                        if (at < kStageCap) mine.gt[at] = compose(key, (uint32_t)i);
                    }
                }
                if (ties) {   // one reservation per wavefront; places past the list's end are only counted
                    uint32_t base = 0;
                    const int leader = __ffsll(ties) - 1;
                    if (lane_id() == leader) base = atomicAdd(&n_tie, (uint32_t)__popcll(ties));
                    const uint32_t at = (uint32_t)__builtin_amdgcn_readlane((int)base, leader) + (uint32_t)__popcll(ties & ((1ull << lane_id()) - 1ull));
                    if (is_tie && at < kStageCap) mine.tie[at] = (uint32_t)i;
                }
            }
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        mine.n_gt = n_gt;
        mine.n_tie = n_tie;
    }
}

// Store into the selection only inside its k words: the positions are sums of counts that other launches left in the
// workspace, and a workspace shared by two overlapping calls (which the boundary forbids) must not turn into a wild
// LDS address.
__device__ __forceinline__ void put_selected(uint64_t* sel, int k, uint32_t e, uint64_t w)
{
    if (e < (uint32_t)k) sel[slot(e)] = w;
}

// One output row: entry gi of the population at rank r of segment `row`'s k.
__device__ __forceinline__ void put_row(int k, uint32_t r, uint32_t gi, const float* __restrict__ score, int32_t* __restrict__ idx_out,
                                        float* __restrict__ val_out, int64_t row, int64_t seg_begin, int64_t seg_end)
{
    if (r < (uint32_t)k) {
        idx_out[row * k + r] = (int32_t)gi;
        if (val_out) val_out[row * k + r] = gi >= seg_begin && gi < seg_end ? score[gi] : 0.f;   // never read outside the segment
    }
}

// The same for a tie, whose score the key T gives without a read (a read in the middle of a run of such rows would
// hold each of them up by a memory round trip); the key of zero stands for two bit patterns and is looked up.
__device__ __forceinline__ void put_tie_row(int k, uint32_t r, uint32_t gi, uint32_t T, const float* __restrict__ score, int32_t* __restrict__ idx_out,
                                            float* __restrict__ val_out, int64_t row, int64_t seg_begin, int64_t seg_end)
{
    if (T == kZeroKey) {
        put_row(k, r, gi, score, idx_out, val_out, row, seg_begin, seg_end);
    } else if (r < (uint32_t)k) {
        idx_out[row * k + r] = (int32_t)gi;
        if (val_out) val_out[row * k + r] = score_of_key(T);
    }
}

// `share` workgroups per segment.  The entries above T need ranking: each workgroup assembles all n_gt of them in
// LDS (the same work, from the same staged lists, the same set of words, in an order that may differ) and then ranks
// and writes the rows of the words whose index hashes to it.  The ties need none: they share the key T, come in
// index order, and the tie of rank r among them owns row n_gt + r; they go from the staged lists (or from a span
// that is read again) straight to the output, each list and each span by one of the workgroups.
__global__ void __launch_bounds__(kSmallThreads) gather_sort_kernel(const float* __restrict__ score, const SegT* __restrict__ segs, int n_seg,
                                                                    int32_t total_blocks, int64_t span, const SelState* __restrict__ state,
                                                                    const Stage* __restrict__ stage, int k, int share,
                                                                    int32_t* __restrict__ idx_out, float* __restrict__ val_out)
{
    __shared__ __align__(16) uint64_t sel[kSelWords];
    __shared__ uint32_t cnt[kSmallThreads];
    __shared__ uint16_t own[PRUNER_MAX_K];   // positions of the words this workgroup ranks
    __shared__ uint32_t n_own;
    __shared__ uint32_t wave_tot[16];
    __shared__ uint32_t tie_buf[kStageCap];
    __shared__ int32_t redo[64];          // workgroups whose span must be read again (list overflow)
    __shared__ uint32_t redo_gt_at[64], redo_tie_before[64];
    __shared__ uint8_t redo_what[64];     // 1: for its entries above T (every workgroup does), 2: for its ties (one does)
    __shared__ uint32_t n_redo, redo_fill;
    __shared__ uint32_t gt_reread;        // a span is read again for its entries above T: their places then differ between workgroups
    __shared__ int32_t partial_block;     // the workgroup in which the tie quota runs out
    __shared__ uint32_t partial_before;
    __shared__ uint32_t first_g[kSmallThreads + 1], first_t[kSmallThreads + 1];   // where each workgroup's lists begin
    __shared__ uint8_t list_skip[kSmallThreads];   // 1: the list of entries above T is not copied, 2: nor the list of ties

    const int s = blockIdx.x / share, part = blockIdx.x % share;
    const SegT seg = segs[s];
    const SelState st = state[2 * n_seg + s];   // as left by the settle launch
    const uint32_t T = st.lowest, k_eq = st.k_rem;
    const uint32_t n_gt = st.n_gt < (uint32_t)k ? st.n_gt : (uint32_t)k;   // (a workspace that overlapping calls share must not turn into wild addresses)
    const int b0 = seg.first_block, b1 = s + 1 < n_seg ? segs[s + 1].first_block : total_blocks;
    if (threadIdx.x == 0) {
        n_redo = 0;
        gt_reread = 0;
        partial_block = -1;
    }
    // (the first batch of list lengths is on its way while the selection is cleared)
    const uint32_t first_cg = b0 + (int)threadIdx.x < b1 ? stage[b0 + threadIdx.x].n_gt : 0u;
    const uint32_t first_ct = b0 + (int)threadIdx.x < b1 ? stage[b0 + threadIdx.x].n_tie : 0u;
    for (int i = threadIdx.x; i < kSelWords; i += kSmallThreads) sel[i] = 0;   // spare words must read as "below everything"
    __syncthreads();

    // Pass over the segment's workgroups in order, kSmallThreads of them at a time: running offsets of both lists.
    // The lists are then copied entry by entry, not list by list: position e finds its list by a search over the
    // offsets, so that all threads copy whatever the lists' lengths (a thread per list would walk the long ones
    // alone).
    uint32_t gt_carry = 0, tie_carry = 0;
    for (int base = b0; base < b1; base += kSmallThreads) {
        const int b = base + threadIdx.x;
        const bool live = b < b1;
        const uint32_t cg = base == b0 ? first_cg : live ? stage[b].n_gt : 0u, ct = base == b0 ? first_ct : live ? stage[b].n_tie : 0u;
        uint32_t tot_g, tot_t;
        const uint32_t at_g = gt_carry + block_excl_scan<kSmallThreads>(cg, wave_tot, &tot_g);
        const uint32_t before_t = tie_carry + block_excl_scan<kSmallThreads>(ct, wave_tot, &tot_t);
        const bool tie_needed = ct > 0 && before_t < k_eq;
        const bool tie_all = tie_needed && before_t + ct <= k_eq;
        const bool over_g = cg > kStageCap, over_t = tie_needed && ct > kStageCap;
        const bool mine = b % share == part;   // this workgroup looks after the ties of that span
        if (live && over_g) gt_reread = 1u;
        if (live && (over_g || (over_t && mine))) {
            const uint32_t slot = atomicAdd(&n_redo, 1u);
            if (slot < 64) {
                redo[slot] = b;
                redo_gt_at[slot] = at_g;
                redo_tie_before[slot] = before_t;
                redo_what[slot] = (uint8_t)((over_g ? 1 : 0) | (over_t && mine ? 2 : 0));
            }
        }
        if (live && tie_needed && !tie_all && !over_t && mine) {
            partial_block = b;       // exactly one workgroup of the launch crosses the quota
            partial_before = before_t;
        }
        first_g[threadIdx.x] = at_g;
        first_t[threadIdx.x] = before_t;
        list_skip[threadIdx.x] = (uint8_t)((over_g ? 1 : 0) | (over_t || !tie_all ? 2 : 0));
        if (threadIdx.x == 0) {
            first_g[kSmallThreads] = gt_carry + tot_g;
            first_t[kSmallThreads] = tie_carry + tot_t;
        }
        __syncthreads();
        // entries above T: position e of the selection is entry e - first_g[j] of the list j with first_g[j] <= e < first_g[j + 1]
        const uint32_t end_g = gt_carry + tot_g;
        for (uint32_t e0 = gt_carry + threadIdx.x; e0 < end_g; e0 += 4 * kSmallThreads) {
            uint64_t w[4];
            bool take[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {   // four loads in flight
                const uint32_t e = e0 + u * kSmallThreads < end_g ? e0 + u * kSmallThreads : end_g - 1;
                int lo = 0;
#pragma unroll
                for (int step = kSmallThreads / 2; step > 0; step >>= 1) lo += first_g[lo + step] <= e ? step : 0;
                const uint32_t i = e - first_g[lo];
                take[u] = e0 + u * kSmallThreads < end_g && (list_skip[lo] & 1) == 0;
                w[u] = stage[base + lo].gt[i < (uint32_t)kStageCap ? i : (uint32_t)kStageCap - 1u];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (take[u]) put_selected(sel, (int)n_gt, e0 + u * kSmallThreads, w[u]);
        }
        // Ties from the lists that are taken whole (the quota does not run out inside them): list j's ties hold the
        // ranks first_t[j] .. first_t[j + 1] - 1 among the segment's ties, in the order of their indices.  A list
        // itself is in no order, so its entries are ranked among themselves, from a copy in LDS behind the entries
        // above T.  The segment's workgroups take turns list by list.
        const uint32_t end_t = tie_carry + tot_t < k_eq ? tie_carry + tot_t : k_eq;
        for (uint32_t r0 = tie_carry + threadIdx.x; r0 < end_t; r0 += 4 * kSmallThreads) {
            uint32_t w[4];
            bool take[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {   // four loads in flight
                const uint32_t r = r0 + u * kSmallThreads < end_t ? r0 + u * kSmallThreads : end_t - 1;
                int lo = 0;
#pragma unroll
                for (int step = kSmallThreads / 2; step > 0; step >>= 1) lo += first_t[lo + step] <= r ? step : 0;
                const uint32_t i = r - first_t[lo];
                take[u] = r0 + u * kSmallThreads < end_t && (list_skip[lo] & 2) == 0 && (base + lo) % share == part && i < (uint32_t)kStageCap;
                w[u] = stage[base + lo].tie[i < (uint32_t)kStageCap ? i : (uint32_t)kStageCap - 1u];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (take[u]) put_selected(sel, k, n_gt + r0 + u * kSmallThreads, (uint64_t)w[u]);
        }
        __syncthreads();
        for (uint32_t r = tie_carry + threadIdx.x; r < end_t; r += kSmallThreads) {
            int lo = 0;
#pragma unroll
            for (int step = kSmallThreads / 2; step > 0; step >>= 1) lo += first_t[lo + step] <= r ? step : 0;
            if ((list_skip[lo] & 2) == 0 && (base + lo) % share == part && n_gt + first_t[lo + 1] <= (uint32_t)k) {
                const uint32_t me = (uint32_t)sel[slot(n_gt + r)];
                uint32_t rank = 0;
                for (uint32_t q = first_t[lo]; q < first_t[lo + 1]; ++q) rank += (uint32_t)sel[slot(n_gt + q)] < me ? 1u : 0u;
                put_tie_row(k, n_gt + first_t[lo] + rank, me, T, score, idx_out, val_out, s, seg.begin, seg.end);
            }
        }
        gt_carry += tot_g;
        tie_carry += tot_t;
        __syncthreads();   // the offsets are rewritten for the next kSmallThreads lists
    }
    __syncthreads();

    // the workgroup where the quota runs out: its smallest indices, by rank among its (at most kStageCap) ties
    if (partial_block >= 0) {
        const Stage& pb = stage[partial_block];
        const uint32_t ct = pb.n_tie < (uint32_t)kStageCap ? pb.n_tie : (uint32_t)kStageCap, want = k_eq - partial_before;
        for (uint32_t i = threadIdx.x; i < ct; i += kSmallThreads) tie_buf[i] = pb.tie[i];
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < ct; i += kSmallThreads) {
            const uint32_t me = tie_buf[i];
            uint32_t rank = 0;
            for (uint32_t j = 0; j < ct; ++j) rank += tie_buf[j] < me ? 1u : 0u;
            if (rank < want) put_tie_row(k, n_gt + partial_before + rank, me, T, score, idx_out, val_out, s, seg.begin, seg.end);
        }
    }
    __syncthreads();

    // overflowed lists: read those spans again, entries above T to their reserved range, ties in index order
    const uint32_t todo = n_redo < 64 ? n_redo : 64;
    for (uint32_t r = 0; r < todo; ++r) {
        const int b = redo[r];
        const bool for_gt = (redo_what[r] & 1) != 0, for_ties = (redo_what[r] & 2) != 0;
        const int64_t lo = seg.begin + (int64_t)(b - b0) * span;
        const int64_t hi = lo + span < seg.end ? lo + span : seg.end;
        if (threadIdx.x == 0) redo_fill = 0;
        __syncthreads();
        uint32_t tie_before = redo_tie_before[r];
        // A wavefront takes kWave * kRedoPer neighbouring entries, lane by lane (coalesced reads): ties keep their index
        // order through counts of comparison masks inside the wavefront and one exchange of the wavefronts' totals per
        // kSmallThreads * kRedoPer entries.
        constexpr int kRedoPer = 16;
        const int lane = lane_id(), wave = threadIdx.x >> 6;
        for (int64_t base = lo; base < hi; base += (int64_t)kSmallThreads * kRedoPer) {
            if (!for_gt && tie_before >= k_eq) break;   // the quota ran out inside this span: nothing more to find
            const int64_t first = base + (int64_t)wave * (kWave * kRedoPer) + lane;
            float val[kRedoPer];   // all loads in flight together (an entry past the end reads the last one and is not used)
#pragma unroll
            for (int j = 0; j < kRedoPer; ++j) val[j] = score[first + j * kWave < hi ? first + j * kWave : hi - 1];
            uint32_t key[kRedoPer];
#pragma unroll
            for (int j = 0; j < kRedoPer; ++j) key[j] = key_of(val[j]);
            if (for_gt) {
#pragma unroll
                for (int j = 0; j < kRedoPer; ++j)
                    if (first + j * kWave < hi && key[j] > T)
                        put_selected(sel, (int)n_gt, redo_gt_at[r] + atomicAdd(&redo_fill, 1u), compose(key[j], (uint32_t)(first + j * kWave)));
            }
            if (for_ties && tie_before < k_eq) {
                uint32_t before_mine[kRedoPer], wave_ties = 0;   // ties of this wavefront before each of this lane's entries
#pragma unroll
                for (int j = 0; j < kRedoPer; ++j) {
                    const unsigned long long m = __ballot(first + j * kWave < hi && key[j] == T);
                    before_mine[j] = wave_ties + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
                    wave_ties += (uint32_t)__popcll(m);
                }
                __syncthreads();  // wave_tot may still be read from an earlier exchange
                if (lane == 0) wave_tot[wave] = wave_ties;
                __syncthreads();
                uint32_t before = 0, all = 0;
#pragma unroll
                for (int w2 = 0; w2 < kSmallThreads / kWave; ++w2) {
                    const uint32_t t = wave_tot[w2];
                    before += w2 < wave ? t : 0u;
                    all += t;
                }
#pragma unroll
                for (int j = 0; j < kRedoPer; ++j) {
                    const uint32_t rank = tie_before + before + before_mine[j];
                    if (first + j * kWave < hi && key[j] == T && rank < k_eq)
                        put_tie_row(k, n_gt + rank, (uint32_t)(first + j * kWave), T, score, idx_out, val_out, s, seg.begin, seg.end);
                }
                tie_before += all;
            }
        }
        __syncthreads();
    }
    if (n_gt == 0) return;
    if (share == 1) {
        finish_segment<kSmallThreads>(sel, (int)n_gt, 0, (int)n_gt, score, idx_out, val_out, s, seg.begin, seg.end, k);
    } else {
        // Which words this workgroup ranks.  Copied from the lists alone, the words have the same places in every
        // workgroup of the segment, and the places are dealt out in turn: no workgroup gets more than the others.
        // Places filled from a span that was read again differ between workgroups; then a hash of the index decides.
        if (threadIdx.x == 0) n_own = 0;
        __syncthreads();
        if (gt_reread == 0) {
            // places part, part + share, ...: no list to build
            const int mine = (int)n_gt > part ? ((int)n_gt - part + share - 1) / share : 0;
            rank_rows<kSmallThreads>(sel, (int)n_gt, nullptr, part, share, mine, cnt, score, idx_out, val_out, s, seg.begin, seg.end, k);
        } else {
            for (int e = threadIdx.x; e < (int)n_gt; e += kSmallThreads) {
                const uint32_t h = (index_of(sel[slot(e)]) * 2654435761u) >> 16;
                if ((int)(h % (uint32_t)share) == part) own[atomicAdd(&n_own, 1u)] = (uint16_t)e;
            }
            __syncthreads();
            rank_rows<kSmallThreads>(sel, (int)n_gt, own, 0, 1, (int)n_own, cnt, score, idx_out, val_out, s, seg.begin, seg.end, k);
        }
    }
}

// ---- pick and levels routes ---------------------------------------------------------------------------------------------
// `share` workgroups per segment.  Each holds what can matter of the segment in registers (sixteen entries per thread), collects all
// entries at or above a bound that at least k entries reach, and ranks those whose index hashes to it among all of them: no lists
// between launches.
//   pick: segments of at most kRow entries are held whole, their first digits counted where they lie; of up to kCountMax, where no maxima
// are asked for (longer ones: pick_long_kernel below).
//   levels: of longer ones blocks of sixteen neighbours are held.  Whoever held the scores left the largest key of every sixteen (and
// of every 64 and 256 where segments are long).  The k best entries lie in the k best blocks (by largest key, then in index order):
// an entry of another block has the largest entries of k blocks before it.  So the k best of the maxima are found, of 256 first,
// then of the 64s in those, then of the sixteens, and the bound that the k-th best maximum gives is one that few more than k entries
// reach: of m maxima in no particular order about m ln(m / (m - k)).  All steps are bounded for any values, ties and sorted
// segments included.
//   A collection that is larger than the limit (ties, entries side by side) is split by up to three digits of the keys' range; ties
// beyond that are written in index order by the segment's first workgroup.
// Bound: the latency of the stages, and what one compute unit draws from beyond its cache: about 50 GB/s, so that a segment of
// 65,536 entries held whole took 5.3 us to arrive; the maxima and blocks of a segment of 50,000, k = 512, are 50 KB.
// Measured, before = digits counted in the draft kernel and segments held whole (above 65,536 a launch that set entries aside first):
// 20 x 50,000, k = 512: draft 13.9 -> 12.8 us, the launch that cleared histograms 2.6 -> none, this one 13.5 -> 14.2; 65,536, k = 128:
// 7.9 -> 7.6, 2.3 -> none, 10.9 -> 9.8; ten segments of 333,333, k = 512: the selection 3 + 7.5 + 8.5 -> 16.5; a kernel of this kind
// is bound by its instructions too (16 wavefronts share four pipes: one more per thread costs 7 ns).
// Good entries side by side make the bound a weak one, and the collection is split: pruner_topk, us by digits and now, 1 x 65,536,
// k = 512, distinct scores 40.5 and 18.4, sorted 38.4 and 25.3, five stretches of good ones 20.9 and 25.5; 1 x 260,000, k = 768, 32.3 and
// 21.4, 32.5 and 37.5, 25.4 and 37.2; 1 x 500,000, k = 512, with ten values 29.9 and 32.5; within one bin 63.4 and 29.6.

constexpr int kPickMax = 65536;
constexpr int kCountMax = 32768;                                // entries held in registers where there are no blocks
constexpr int kXcds = 8;                                        // parts of the device with a cache of their own; workgroups go to them in turn
constexpr int kPickCap = 8192;                                  // words a workgroup collects
constexpr int kPickWords = kPickCap + kPickCap / 32 + 4;
constexpr int kLevelK = 1024;                                   // blocks of sixteen that registers hold
constexpr int kLevelMostK = kLevelK / 4 * 3;                    // a larger k leaves the bound so little room that it takes every digit: the filter of 400,000, k = 768,
                                                                // 26.4 us (27 by digits and lists), k = 1,000 39 (27); of 3,000,000 43 (48) and 61 (49); 10 x 300,001 62 (62) and 72 (62)
static_assert(kLevelK * 16 == kRow, "selected blocks are held as a short segment is");
constexpr int kDirectBlocks = 16384;                             // up to here all maxima of a level are looked at, above it those in the best of the next
constexpr int64_t kLevelMax = 256 * (int64_t)kDirectBlocks;     // three levels at most, the top one held.  The filter of 4 M, k = 512, 44 us (51 by digits), of 9.3 M 107 (93; 92 by
                                                                // the blocks of 256)
// What is collected is ranked word against word, so it has to be little more than k: otherwise the bin is split first (two
// values shared by 20,000 entries, k = 512: 84 us with all of the bin ranked, 25 with the limit).
__host__ __device__ constexpr int collect_limit(int k) { return k + k / 4 + 256; }
static_assert(kPickCap >= collect_limit(PRUNER_MAX_K), "a collection fits");

// A round of ranking (64 words against all n) takes about n / 750 us, a sort of P words by a workgroup P / 230.
constexpr int kSortFactor = 3;   // rounds x n beyond this many times P: sort
constexpr int kTrimMax = 512;
static_assert(kTrimMax <= kBigThreads, "a word of the last bin per thread");

// The lists route: at most 32 spans per segment, so that a segment that has to be gone through again by one workgroup is still
// a matter of microseconds.
constexpr int64_t kListsMax = 32 * (int64_t)kRow;
constexpr int kListCap = 1280;
struct List {                 // the entries of one span at or above the bin (lies in the span's Stage)
    uint32_t count, pad;      // may exceed the capacity
    uint64_t word[kListCap];  // in no order; where there are NaN, some below the bin may be among them, and of a span that has more than
                              // these at or above the bin, its own k best at least
};
static_assert(sizeof(List) <= sizeof(Stage), "a list lies where the spans route keeps its stage");

// A thread's sixteen entries of a sweep as a mask (bit j: entry j is not below t0, which a NaN never is: the mask holds every entry
// whose key is at or above t0's and, where there are NaN, some others; whoever needs exactly those looks at the keys).
__device__ __forceinline__ uint32_t mask_of_sweep(const float (&val)[kBigPer], float t0, int64_t row, int64_t hi)
{
    uint32_t mask = 0;
#pragma unroll
    for (int j = kBigPer - 1; j >= 0; --j) mask = 2 * mask + (val[j] < t0 ? 0u : 1u);
    if (row + kRow > hi) {   // the last sweep: entries past the end (read as 0) are none
#pragma unroll
        for (int j = 0; j < kBigPer; ++j) mask &= sweep_index(row, j) < hi ? ~0u : ~(1u << j);
    }
    return mask;
}
// A score that nothing with a key at or above `key` is below (a key beyond the infinities' names a NaN: then no number is below).
__device__ __forceinline__ float threshold_of(uint32_t key)
{
    const float t = score_of_key(key);
    return t != t ? -__builtin_inff() : t;
}
// Consecutive places of a list for the `mine` entries of each thread: the wavefront's threads share out what one reserves.
__device__ __forceinline__ uint32_t reserve(uint32_t* fill, uint32_t mine)
{
    const uint32_t upto = wave_inclusive_sum(mine);
    uint32_t base = 0;
    if (lane_id() == kWave - 1 && upto) base = atomicAdd(fill, upto);
    return (uint32_t)__builtin_amdgcn_readlane((int)base, kWave - 1) + upto - mine;
}

// The least and the largest key of the bin lowest .. lowest + width among what the workgroup's threads saw, in two LDS words that
// start as 0 (the least as its complement): a bin that holds one value only, as those of measured copies do, is then known for
// it and is not split digit by digit.
__device__ __forceinline__ void note_range(uint32_t not_least, uint32_t largest, uint32_t* range)
{
#pragma unroll
    for (int step = 1; step < kWave; step *= 2) {
        const uint32_t a = __shfl_xor(not_least, step), b = __shfl_xor(largest, step);
        not_least = a > not_least ? a : not_least;
        largest = b > largest ? b : largest;
    }
    if (lane_id() == 0 && (not_least | largest) != 0u) {
        atomicMax(&range[0], not_least);
        atomicMax(&range[1], largest);
    }
}

// The list of a span that has more at or above the bin than it holds: the span's own k best, for whatever is among the segment's k
// best is among these.  They are found as the segment's are, digit by digit in the bin; ties that are too many are taken in
// index order.  (Scores within one bin, 480,000 in one segment, k = 76: the workgroups that collect took 120 us going through
// the spans of all lists themselves, the call takes 51 now, 52 by the spans route.)  A function of its own: list_kernel
// as a rule does without it and keeps its registers.
__device__ __attribute__((noinline)) void own_best(const float* __restrict__ span_score, int span_len, uint32_t first_index, int k, uint32_t lowest, uint32_t width,
                                                   uint32_t* hist, uint32_t* wave_tot, uint32_t* found, uint32_t* fill, uint32_t* range, List* mine_list)
{
    List& mine = *mine_list;
    uint32_t lo_key = lowest, w = width, rem = (uint32_t)k, in_bin = 0;
    float val[kBigPer];
    bool all = false;   // (with NaN below the bin in the list: the rest may fit after all)
#pragma unroll 1
    for (int digits = 0; digits < 3; ++digits) {
        const int sh = next_shift(w);
        __syncthreads();
        for (int i = threadIdx.x; i < kBins; i += kBigThreads) hist[i] = 0;
        if (threadIdx.x == 0) *fill = range[0] = 0;
        __syncthreads();
        uint32_t above = 0, inside = 0;   // of this thread
#pragma unroll 1
        for (int row = 0; row < span_len; row += kRow) {
            load_sweep(span_score, row, span_len, val);
#pragma unroll
            for (int j = 0; j < kBigPer; ++j) {
                const uint32_t key = key_of(val[j]);
                const bool there = (int)sweep_index(0, j) < span_len - row, in = there && key - lo_key <= w;
                if (in) atomicAdd(&hist[(key - lo_key) >> sh], 1u);
                inside += in ? 1u : 0u;
                above += there && key > lo_key && !in ? 1u : 0u;
            }
        }
        if (digits == 0) {
            if (above) atomicAdd(fill, above);
            if (inside) atomicAdd(&range[0], inside);
        }
        __syncthreads();
        if (digits == 0) {
            all = *fill + range[0] <= (uint32_t)kListCap;
            if (all) break;
            rem = (uint32_t)k - *fill;   // (fewer than k lie above the segment's bin)
        }
        find_bucket(hist, rem, wave_tot, found);
        lo_key += found[0] << sh;
        w = (1u << sh) - 1u;
        rem = found[1];
        in_bin = found[2];
        if ((uint32_t)k - rem + in_bin <= (uint32_t)kListCap || w == 0u) break;
    }
    const bool ties_apart = !all && (uint32_t)k - rem + in_bin > (uint32_t)kListCap;
    __syncthreads();
    if (threadIdx.x == 0) *fill = 0;
    __syncthreads();
    uint32_t ties_before = 0;
#pragma unroll 1
    for (int row = 0; row < span_len; row += kRow) {
        load_sweep(span_score, row, span_len, val);
        uint32_t mask = 0;
#pragma unroll
        for (int j = 0; j < kBigPer; ++j) {
            const uint32_t key = key_of(val[j]);
            mask |= (int)sweep_index(0, j) < span_len - row && (ties_apart ? key > lo_key : key >= lo_key) ? 1u << j : 0u;
        }
        uint32_t at = reserve(fill, (uint32_t)__popc(mask));
        for (; mask; mask &= mask - 1, ++at) {
            const int i = (int)sweep_index(row, __ffs(mask) - 1);
            if (at < (uint32_t)kListCap) mine.word[at] = compose(key_of(span_score[i]), first_index + (uint32_t)i);
        }
        if (ties_apart && ties_before < rem) {
            // behind the k - rem above them, numbered in index order: four neighbours of every thread at a time
#pragma unroll
            for (int q = 0; q < kBigPer / 4; ++q) {
                uint32_t tie = 0, total;
#pragma unroll
                for (int e = 0; e < 4; ++e) tie |= (int)sweep_index(0, 4 * q + e) < span_len - row && key_of(val[4 * q + e]) == lo_key ? 1u << e : 0u;
                uint32_t number = ties_before + block_excl_scan<kBigThreads>((uint32_t)__popc(tie), wave_tot, &total);
                for (; tie && number < rem; tie &= tie - 1, ++number)
                    mine.word[(uint32_t)k - rem + number] = compose(lo_key, first_index + (uint32_t)sweep_index(row, 4 * q + __ffs(tie) - 1));
                ties_before += total;
            }
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) mine.count = ties_apart ? (uint32_t)k : *fill;
}

__global__ void __launch_bounds__(kBigThreads) __attribute__((amdgpu_waves_per_eu(8))) list_kernel(const float* __restrict__ score, const SegT* __restrict__ segs, int n_seg,
                                                                                                    int64_t span, int R, int k,
                                                                                                    const uint32_t* __restrict__ ghist0,
                                                                                                    uint32_t* __restrict__ ghist1, uint32_t* __restrict__ granges,
                                                                                                    Stage* __restrict__ stage)
{
    __shared__ uint32_t hist[kBins];
    __shared__ uint32_t wave_tot[16];
    __shared__ uint32_t found[3];
    __shared__ uint32_t range[2];
    __shared__ uint32_t fill;
    const int s = segment_of_block(segs, n_seg, blockIdx.x);
    const SegT seg = segs[s];
    const int64_t lo = seg.begin + (int64_t)(blockIdx.x - seg.first_block) * span;
    const int64_t hi = lo + span < seg.end ? lo + span : seg.end;
    float val[kBigPer];
    load_sweep(score, lo, hi, val);   // the first sweep travels while the bin is looked up
    bucket_of_pass<8>(ghist0, R, n_seg, s, (uint32_t)k, hist, wave_tot, found);
    uint32_t lowest, width;
    first_digit_range(found[0], lowest, width);
    const float t0 = threshold_of(lowest);
    const int shift = next_shift(width);
    const uint32_t at_or_above = (uint32_t)k - found[1] + found[2];   // of the bin, in the segment
    const bool crowded = at_or_above > (uint32_t)collect_limit(k);    // the second digit will be asked for
    __syncthreads();
    if (threadIdx.x == 0) fill = range[0] = range[1] = 0;
    if (crowded)
        for (int i = threadIdx.x; i < kBins; i += kBigThreads) hist[i] = 0;
    __syncthreads();
    List& mine = *reinterpret_cast<List*>(&stage[blockIdx.x]);
    uint32_t not_least = 0, largest = 0;
    for (int64_t row = lo; row < hi; row += kRow) {
        if (row > lo) load_sweep(score, row, hi, val);
        uint32_t mask = mask_of_sweep(val, t0, row, hi);
        if (crowded) {
#pragma unroll
            for (int j = 0; j < kBigPer; ++j) {
                const uint32_t key = key_of(val[j]);
                const bool in = ((mask >> j) & 1u) != 0u && key - lowest <= width;
                light_hist_add(hist, (key - lowest) >> shift, in);
                not_least = in && ~key > not_least ? ~key : not_least;
                largest = in && key > largest ? key : largest;
            }
        }
        uint32_t at = reserve(&fill, (uint32_t)__popc(mask));
        while (mask) {
            const int64_t i = sweep_index(row, __ffs(mask) - 1);
            mask &= mask - 1;
            if (at < (uint32_t)kListCap) mine.word[at] = compose(key_of(score[i]), (uint32_t)i);
            else break;   // (the count says that there are more)
            ++at;
        }
    }
    if (crowded) note_range(not_least, largest, range);
    __syncthreads();
    if (threadIdx.x == 0) mine.count = fill;
    if (crowded) {
        flush_hist<kBigThreads>(hist, ghist1, 1, n_seg, s);
        if (threadIdx.x < 2 && range[threadIdx.x] != 0u) atomicMax(&granges[(size_t)s * kBins + threadIdx.x], range[threadIdx.x]);
    }
    // (k up to kLevelMostK comes here from pruner_topk_static only, which has no room for maxima.)
    // One value: its ties need no list.  Fewer spans' worth of such entries (a sorted segment; a shorter one): whoever collects goes
    // through those spans in less time than this takes, 10 to 20 us (within one bin, k = 90: 1 x 200,000 70 -> 49 us, 1 x 350,000
    // 96 -> 51; k = 512 or 686: 8 x 220,000 50 -> 60, 3 x 274,000 50 -> 61, 3 x 350,000 103 -> 69).
    if (fill > (uint32_t)kListCap && k <= kListCap && crowded && at_or_above > (k <= 128 ? 12u : 18u) * (uint32_t)span && ~range[0] != range[1])
        own_best(score + lo, (int)(hi - lo), (uint32_t)lo, k, lowest, width, hist, wave_tot, found, &fill, range, &mine);
}

// The n words in sel to the rows (those below row_len = k) of one segment: ranked in rounds of 64 per workgroup, the words shared out over the
// segment's workgroups, or sorted, all of them by every workgroup, whatever costs less (see kSortFactor).
// SORT: with the way of sorting (the other calls' kernel is shorter without it).  k_rem of the words with keys lowest .. lowest + width
// are selected, and all above; exact: these two facts are, and no word lies below, so that the sort may leave the surplus out.  same_places: the words lie in the same
// places in every workgroup, which are dealt out in turn (by the hash some have half as many again as others, and with them a round more:
// 5,179 words, 128 workgroups, 40 each: 23.5 us, dealt out 15.0).
template <bool SORT>
__device__ __forceinline__ void write_collection(uint64_t* sel, uint32_t* place, uint32_t* cnt, uint32_t* fill, uint32_t* n_own, int n, int k, int share, int part,
                                                 uint32_t k_rem, uint32_t lowest, uint32_t width, bool exact, const float* __restrict__ score,
                                                 int32_t* __restrict__ idx_out, float* __restrict__ val_out, int s, const SegT& seg, bool same_places = false)
{
    uint16_t* own = reinterpret_cast<uint16_t*>(place);
    const int n_last = n - (int)((uint32_t)k - k_rem);   // the words of the last bin
    const bool trim = exact && n > k && n_last <= kTrimMax && pow2_at_least(n) > pow2_at_least(k);
    const int rounds = (n + 64 * share - 1) / (64 * share);
    if (SORT && rounds * n > kSortFactor * pow2_at_least(trim ? k : n)) {
        if (trim) {
            // the sort is half as long without those of the last bin that are not selected: their places go to what lies behind k
            uint64_t* bin_word = reinterpret_cast<uint64_t*>(place);
            uint16_t *bin_at = reinterpret_cast<uint16_t*>(place + 2 * kTrimMax), *hole = bin_at + kTrimMax;
            static_assert(kPickCap * sizeof(uint32_t) >= kTrimMax * (sizeof(uint64_t) + 2 * sizeof(uint16_t)), "the lists fit");
            __syncthreads();
            if (threadIdx.x == 0) *fill = 0;
            __syncthreads();
            for (int e = threadIdx.x; e < n; e += kBigThreads) {
                const uint64_t w = sel[slot((uint32_t)e)];
                if ((uint32_t)(w >> 32) - lowest <= width) {
                    const uint32_t at = atomicAdd(fill, 1u);
                    if (at < (uint32_t)kTrimMax) bin_word[at] = w, bin_at[at] = (uint16_t)e;
                }
            }
            __syncthreads();
            if ((int)threadIdx.x < n_last) {
                const uint64_t me = bin_word[threadIdx.x];
                const int at = bin_at[threadIdx.x];
                uint32_t better = 0;
                for (int x = 0; x < n_last; ++x) better += bin_word[x] > me ? 1u : 0u;
                if (better >= k_rem) {
                    sel[slot((uint32_t)at)] = 0;
                    if (at < k) hole[atomicAdd(n_own, 1u)] = (uint16_t)at;
                }
            }
            if (threadIdx.x == 0) *fill = 0;
            __syncthreads();
            for (int e = k + (int)threadIdx.x; e < n; e += kBigThreads) {
                const uint64_t w = sel[slot((uint32_t)e)];
                if (w != 0ull) sel[slot(hole[atomicAdd(fill, 1u)])] = w;
            }
            __syncthreads();
            n = k;
        }
        const int rows = n < k ? n : k, per = (rows + share - 1) / share, lo = part * per < rows ? part * per : rows;   // each writes its part of the rows
        finish_segment<kBigThreads>(sel, n, lo, lo + per < rows ? lo + per : rows, score, idx_out, val_out, s, seg.begin, seg.end, k);
        n = 0;
    }
    if (same_places) {
        __syncthreads();
        if (n > 0) rank_rows<kBigThreads>(sel, n, nullptr, part, share, n > part ? (n - part + share - 1) / share : 0, cnt, score, idx_out, val_out, s, seg.begin, seg.end, k);
        return;
    }
    // (every workgroup has its own order of the words: a hash of the index decides who ranks a word)
    for (int e = threadIdx.x; e < n; e += kBigThreads) {
        const uint32_t h = (index_of(sel[slot((uint32_t)e)]) * 2654435761u) >> 16;
        if ((int)(h % (uint32_t)share) == part) own[atomicAdd(n_own, 1u)] = (uint16_t)e;
    }
    __syncthreads();
    if (n > 0) rank_rows<kBigThreads>(sel, n, own, 0, 1, (int)*n_own, cnt, score, idx_out, val_out, s, seg.begin, seg.end, k);
}

// Four neighbouring maxima from number `at` on, 0 for those past the last.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 u32x4_a4 __attribute__((aligned(4)));
__device__ __forceinline__ u32x4 maxima_at(const uint32_t* maxima, int at, int n)
{
    u32x4 w = *reinterpret_cast<const u32x4_a4*>(maxima + at);
#pragma unroll
    for (int e = 1; e < 4; ++e) w[e] = at + e < n ? w[e] : 0u;
    return w;
}
// The blocks whose maxima reach a bound that at least k of them reach, at most kLevelK, in index order, in `out`; the bound is
// returned.  Where more reach it, it is raised digit by digit, and of maxima that all equal it the first ones are taken.
// parents (n_parents > 0): only the blocks that these numbers, in order, name four each, and `bound` is one that k of them reach; else 0.  All threads of the workgroup; hist,
// wave_tot, found, range: its LDS.  (The loops are kept rolled: a workgroup runs this once or twice, and what unrolled code costs is its
// way into the instruction cache.)
__device__ __forceinline__ uint32_t best_blocks(const uint32_t* __restrict__ maxima, int n, const uint32_t* parents, int n_parents, uint32_t bound, uint32_t k, uint32_t* hist,
                                                uint32_t* wave_tot, uint32_t* found, uint32_t* range, uint32_t* out, int* n_out)
{
    // Quads of maxima per thread and row, neighbours: the order of the threads is that of the blocks.
    constexpr int kQuads = 4;
    const int n_quads = n_parents > 0 ? n_parents : (n + 3) >> 2;
    const int of = n_quads > 3 * kBigThreads ? 4 : n_quads > 2 * kBigThreads ? 3 : n_quads > kBigThreads ? 2 : 1, rows = (n_quads + of * kBigThreads - 1) / (of * kBigThreads);
    auto first = [&](int q) -> int { return n_parents > 0 ? 4 * (int)parents[q] : 4 * q; };
    uint32_t v[4 * kQuads], held = 0;   // held: the maxima among them, as bits
    int n_mine = 0;                     // quads of this thread
    auto load = [&](int row) {
        const int q0 = (row * kBigThreads + (int)threadIdx.x) * of;
        n_mine = n_quads - q0 < of ? n_quads - q0 : of;
        u32x4 w[kQuads];
#pragma unroll
        for (int j = 0; j < kQuads; ++j)
            if (j < of) w[j] = maxima_at(maxima, first(q0 + j < n_quads ? q0 + j : n_quads - 1), n);
#pragma unroll
        for (int j = 0; j < kQuads; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) v[4 * j + e] = j < of && j < n_mine ? w[j][e] : 0u;
        held = maxima_held(n_mine, first(q0 + n_mine - 1), n);   // (without quads: n_quads - 1, which is there)
    };
    if (rows == 1) load(0);
    // maxima of sixteen and of four of the maxima serve as well where there are enough of them
    int together = of == 4 && n_quads >= 16 * (int)k ? 16 : n_quads >= 4 * (int)k ? 4 : 1;
    uint32_t lowest = bound, width = ~0u - bound, k_rem = k, in_bin = 0, taken = 0, largest = 0;
#pragma unroll 1
    for (int attempt = 0; attempt < 2; ++attempt) {
        // first: the bin of k maxima, split once where it holds many (among the parts of blocks chosen already their bound does as
        // well); again, from that bound on and with every block's own, where more than kLevelK blocks reach it
        const uint32_t enough = attempt == 0 ? (uint32_t)collect_limit((int)k) : (uint32_t)kLevelK;
#pragma unroll 1
        for (int digit = 0; digit < (attempt == 0 ? (n_parents > 0 ? 0 : 2) : 3) && width != 0u; ++digit) {
            const bool narrow_bins = attempt == 0 && digit == 0;
            const int shift = next_shift(width);
            __syncthreads();
            for (int i = threadIdx.x; i < kBins; i += kBigThreads) hist[i] = 0;
            __syncthreads();
            auto add = [&](uint32_t key, bool there) {
                const uint32_t digit = narrow_bins ? first_digit_of(key) : (key - lowest) >> shift;
                const bool counts = there && key >= lowest && key - lowest <= width;
                if (of > 1) light_hist_add(hist, digit, counts);
                else if (counts) atomicAdd(&hist[digit], 1u);   // (few: also where they queue on one address)
            };
#pragma unroll 1
            for (int row = 0; row < rows; ++row) {
                if (rows > 1) load(row);
                uint32_t best = 0;
#pragma unroll
                for (int j = 0; j < kQuads; ++j) {
                    if (j >= of) continue;
                    if (together == 1) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) add(v[4 * j + e], j < n_mine);
                    } else {
                        const uint32_t a = v[4 * j] > v[4 * j + 1] ? v[4 * j] : v[4 * j + 1], b = v[4 * j + 2] > v[4 * j + 3] ? v[4 * j + 2] : v[4 * j + 3];
                        const uint32_t top = a > b ? a : b;
                        if (together == 4) add(top, j < n_mine);
                        else best = top > best ? top : best;
                    }
                }
                if (together == 16) add(best, n_mine > 0);
            }
            __syncthreads();
            find_bucket(hist, k_rem, wave_tot, found);
            if (narrow_bins) {
                first_digit_range(found[0], lowest, width);
            } else {
                lowest += found[0] << shift;
                width = (1u << shift) - 1u;
                width = attempt == 1 && largest - lowest < width ? largest - lowest : width;
            }
            k_rem = found[1];
            in_bin = found[2];
            if (k - k_rem + in_bin <= enough) break;
        }
        // the blocks at or above the bound (ties apart: above it, and the first k_rem that equal it), in order
        const bool ties_apart = attempt == 1 && k - k_rem + in_bin > (uint32_t)kLevelK;
        uint32_t ties_before = 0, total;
        taken = 0;
#pragma unroll 1
        for (int row = 0; row < rows; ++row) {
            if (rows > 1) load(row);
            uint32_t mask = 0, equal = 0;
#pragma unroll
            for (int j = 0; j < kQuads; ++j) {
                if (j >= of) continue;
#pragma unroll
                for (int e = 0; e < 4; ++e) mask |= v[4 * j + e] >= lowest ? 1u << (4 * j + e) : 0u;
            }
            mask &= held;
            if (ties_apart) {
#pragma unroll
                for (int j = 0; j < 4 * kQuads; ++j) equal |= v[j] == lowest ? 1u << j : 0u;
                equal &= held;
                mask ^= equal;
                uint32_t number = ties_before + block_excl_scan<kBigThreads>((uint32_t)__popc(equal), wave_tot, &total);
#pragma unroll 1
                for (; equal && number < k_rem; equal &= equal - 1u, ++number) mask |= equal & (0u - equal);
                ties_before += total;
            }
            uint32_t at = taken + block_excl_scan<kBigThreads>((uint32_t)__popc(mask), wave_tot, &total);
#pragma unroll 1
            for (; mask; mask &= mask - 1u, ++at) {
                const int j = __ffs((int)mask) - 1;
                if (at < (uint32_t)kLevelK) out[at] = (uint32_t)(first((row * kBigThreads + (int)threadIdx.x) * of + (j >> 2)) + (j & 3));
            }
            taken += total;
        }
        if (taken <= (uint32_t)kLevelK || attempt == 1) break;
        // (a range that holds one key only is known for it and not split)
        if (threadIdx.x == 0) range[0] = range[1] = 0;
        __syncthreads();
        uint32_t not_least = 0;
#pragma unroll 1
        for (int row = 0; row < rows; ++row) {
            if (rows > 1) load(row);
#pragma unroll
            for (int j = 0; j < 4 * kQuads; ++j) {
                const bool in = ((held >> j) & 1u) != 0u && v[j] >= lowest;
                not_least = in && ~v[j] > not_least ? ~v[j] : not_least;
                largest = in && v[j] > largest ? v[j] : largest;
            }
        }
        note_range(not_least, largest, range);
        __syncthreads();
        lowest = ~range[0];
        largest = range[1];
        width = largest - lowest;
        together = 1;
        k_rem = k;
        in_bin = taken;
    }
    __syncthreads();
    if (threadIdx.x == 0) range[0] = range[1] = 0;
    *n_out = (int)(taken < (uint32_t)kLevelK ? taken : (uint32_t)kLevelK);
    return lowest;
}

// The largest keys of every 16, 64 and 256 neighbouring entries; the latter two may be null where no segment has more than
// kDirectBlocks blocks of 16 (of 64).
struct Maxima {
    const uint32_t *of16, *of64, *of256;
};

// LEVELS: segments longer than kRow, by blocks.  ghist0 (or null): the first digits' histogram, in R copies.
template <bool LEVELS, bool SORT, class Table>
__global__ void __launch_bounds__(kBigThreads) pick_kernel(const float* __restrict__ score, Table segs, int n_seg, int n_total, int k, int share,
                                                           Maxima maxima, const uint32_t* __restrict__ ghist0, int R, int32_t* __restrict__ idx_out,
                                                           float* __restrict__ val_out)
{
    constexpr int kQ = (LEVELS ? kRow : kCountMax) / (4 * kBigThreads);
    __shared__ __align__(16) uint64_t sel[kPickWords];
    __shared__ __align__(16) uint32_t place[kPickCap];   // selected blocks of the level before; then indices inside the segment; then which words this workgroup ranks
    __shared__ uint32_t hist[kBins];          // later: the ranking's counts
    __shared__ uint32_t blocks[LEVELS ? kLevelK : 1];
    __shared__ uint32_t wave_tot[16];
    __shared__ uint32_t found[3];
    __shared__ uint32_t fill, n_own, range[2];
    // The workgroups of a segment go to one of the eight parts of the device: its cache then reads the segment once for all.
    const int per_xcd = (n_seg * share + kXcds - 1) / kXcds, job = (int)(blockIdx.x % kXcds) * per_xcd + (int)(blockIdx.x / kXcds);
    if (job >= n_seg * share) return;
    const int s = job / share, part = job % share;
    const SegT seg = segs.at(s);
    const int len = (int)(seg.end - seg.begin);
    const float* seg_score = score + seg.begin;

    int n_blocks = 0;
    uint32_t lowest = 0, width = ~0u, k_rem = (uint32_t)k, in_bin = 0;
    const bool whole = !LEVELS || len <= kRow;
    if (!whole) {
        const int n16 = (len + 15) >> 4, n64 = (len + 63) >> 6;
        const int top = n16 <= kDirectBlocks ? 0 : n64 <= kDirectBlocks ? 1 : 2;
#pragma unroll 1
        for (int level = top; level >= 0; --level) {
            if (level < top) {
                for (int i = threadIdx.x; i < n_blocks; i += kBigThreads) place[i] = blocks[i];
                __syncthreads();
            }
            const uint32_t* const of = level == 0 ? maxima.of16 + block16_slot(seg.begin, s) : level == 1 ? maxima.of64 + block64_slot(seg.begin, s) : maxima.of256 + block_max_slot(seg.begin, s);
            lowest = best_blocks(of, level == 0 ? n16 : level == 1 ? n64 : (len + 255) >> 8, place, level < top ? n_blocks : 0, lowest, (uint32_t)k, hist, wave_tot, found, range, blocks, &n_blocks);
        }
        width = ~0u - lowest;
    }

    // Groups of four neighbours, at multiples of four from the segment's begin: kQ per thread and row.
    const int last = n_total - 4 - (int)seg.begin;   // (there are more than four scores in all)
    const int held = whole ? len : 16 * n_blocks, rows = (held + kQ * 4 * kBigThreads - 1) / (kQ * 4 * kBigThreads);
    auto group_begin = [&](int g) -> int {
        const int at = g * kBigThreads + (int)threadIdx.x;
        if (!LEVELS || whole) return 4 * at;
        return (at >> 2) < n_blocks ? (int)(16u * blocks[at >> 2]) + 4 * (at & 3) : len;
    };
    // (a group that would reach past the end of the scores starts earlier: there_of tells which of the four are the group's)
    auto load_group = [&](int i) { return f32x4(*reinterpret_cast<const f32x4_a4*>(seg_score + (i < last ? i : last))); };
    auto there_of = [&](int i) -> uint32_t {
        const int left = len - i, moved = i < last ? 0 : i - last;
        return left <= 0 ? 0u : ((left < 4 ? (1u << left) - 1u : 15u) << moved) & 15u;
    };
    f32x4 row_of[kQ];
    auto load_row = [&](int row) {
#pragma unroll
        for (int q = 0; q < kQ; ++q)
            if ((kQ * row + q) * 4 * kBigThreads < held) row_of[q] = load_group(group_begin(kQ * row + q));
    };
    auto each_key = [&](auto&& what) {   // what(index, key, whether it is the segment's); a single row is read once
#pragma unroll 1
        for (int row = 0; row < rows; ++row) {
            if (rows > 1) load_row(row);
#pragma unroll
            for (int q = 0; q < kQ; ++q) {
                if ((kQ * row + q) * 4 * kBigThreads >= held) continue;
                const int i = group_begin(kQ * row + q);
                const uint32_t there = there_of(i);
                uint32_t keys[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) keys[e] = key_of(row_of[q][e]);
                what(i < last ? i : last, keys, there);
            }
        }
    };
    if (rows == 1) load_row(0);
    // (every group that is held is held whole: the segment's end lies in none of them)
    const bool all_whole = whole || (len & 15) == 0 || blocks[n_blocks - 1] != (uint32_t)(len >> 4);
    const uint32_t limit = (uint32_t)collect_limit(k);
    bool exact = whole;   // k_rem, in_bin: of the bin lowest .. lowest + width, by count
    if (whole) {
        if (ghist0) {
            bucket_of_pass<8>(ghist0, R, n_seg, s, (uint32_t)k, hist, wave_tot, found);
        } else {
            for (int i = threadIdx.x; i < kBins; i += kBigThreads) hist[i] = 0;
            __syncthreads();
            each_key([&](int, const uint32_t (&keys)[4], uint32_t there) {
#pragma unroll
                for (int e = 0; e < 4; ++e) light_hist_add(hist, first_digit_of(keys[e]), ((there >> e) & 1u) != 0u);
            });
            __syncthreads();
            find_bucket(hist, (uint32_t)k, wave_tot, found);
        }
        first_digit_range(found[0], lowest, width);
        k_rem = found[1];
        in_bin = found[2];
    }
    if (threadIdx.x == 0) fill = n_own = range[0] = range[1] = 0;
    __syncthreads();
    bool ties_apart = false;
#pragma unroll 1
    for (int attempt = 0; attempt < 2; ++attempt) {
        if ((uint32_t)k - k_rem + in_bin > limit && !ties_apart) {
            // Too many (ties, entries side by side).  The bound is raised digit by digit; a range that holds one key only is known for it
            // and not split.
            uint32_t not_least = 0, largest = 0;
            each_key([&](int, const uint32_t (&keys)[4], uint32_t there) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const bool in = ((there >> e) & 1u) != 0u && keys[e] >= lowest && keys[e] - lowest <= width;
                    not_least = in && ~keys[e] > not_least ? ~keys[e] : not_least;
                    largest = in && keys[e] > largest ? keys[e] : largest;
                }
            });
            note_range(not_least, largest, range);
            __syncthreads();
            largest = range[1];
            lowest = ~range[0];
            width = largest - lowest;
            exact = true;
#pragma unroll 1
            for (int digits = 0; digits < 3 && width != 0u && (uint32_t)k - k_rem + in_bin > limit; ++digits) {   // (32 bits at most)
                const int shift = next_shift(width);
                for (int i = threadIdx.x; i < kBins; i += kBigThreads) hist[i] = 0;
                __syncthreads();
                each_key([&](int, const uint32_t (&keys)[4], uint32_t there) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) light_hist_add(hist, (keys[e] - lowest) >> shift, ((there >> e) & 1u) != 0u && keys[e] >= lowest && keys[e] - lowest <= width);
                });
                __syncthreads();
                find_bucket(hist, k_rem, wave_tot, found);
                lowest += found[0] << shift;
                width = (1u << shift) - 1u;
                width = largest - lowest < width ? largest - lowest : width;
                k_rem = found[1];
                in_bin = found[2];
                __syncthreads();
            }
            ties_apart = (uint32_t)k - k_rem + in_bin > limit;
        }
        // the places of the entries at or above the bound (ties apart: above it).  (Words straight out of the registers, sixteen stores
        // under a condition each, took 2 us more than the places and the second look at the scores.)  At first by comparison: what is
        // not below includes every NaN, which the ranking then orders by its bits, unless that makes too many.
        const uint32_t expected = ties_apart ? (uint32_t)k - k_rem : (uint32_t)k - k_rem + in_bin;
        const float t0 = threshold_of(ties_apart ? lowest + 1u : lowest);
#pragma unroll 1
        for (int row = 0; row < rows; ++row) {
            if (rows > 1) load_row(row);
            uint32_t mask = 0;   // bit 4 q + e
            if (attempt == 0) {
#pragma unroll
                for (int q = kQ - 1; q >= 0; --q) {
                    uint32_t four = 0;
                    if ((kQ * row + q) * 4 * kBigThreads < held) {
#pragma unroll
                        for (int e = 3; e >= 0; --e) four = 2u * four + (row_of[q][e] < t0 ? 0u : 1u);
                        if (!all_whole || (kQ * row + q + 1) * 4 * kBigThreads > held) four &= there_of(group_begin(kQ * row + q));
                    }
                    mask = 16u * mask + four;
                }
            } else {
#pragma unroll
                for (int q = 0; q < kQ; ++q) {
                    if ((kQ * row + q) * 4 * kBigThreads >= held) continue;
                    uint32_t four = 0;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const uint32_t key = key_of(row_of[q][e]);
                        four |= key > lowest || (!ties_apart && key == lowest) ? 1u << e : 0u;
                    }
                    mask |= (four & there_of(group_begin(kQ * row + q))) << (4 * q);
                }
            }
            uint32_t to = reserve(&fill, (uint32_t)__popc(mask));
#pragma unroll 1
            for (; mask; mask &= mask - 1u, ++to) {
                const int bit = __ffs((int)mask) - 1, i = group_begin(kQ * row + (bit >> 2));
                if (to < (uint32_t)kPickCap) place[to] = (uint32_t)((i < last ? i : last) + (bit & 3));
            }
        }
        __syncthreads();
        const uint32_t collected = fill;
        if (exact ? collected == expected : collected <= limit) break;
        __syncthreads();
        if (threadIdx.x == 0) fill = 0;
        __syncthreads();   // (what is known by count is collected again at once)
        if (!exact) in_bin = collected;
    }
    if (ties_apart && part == 0) {
        // ties, all of the key `lowest`, in index order: the tie of rank r owns row k - k_rem + r (groups and threads are in that order)
        uint32_t before = 0;
#pragma unroll 1
        for (int g = 0; g * 4 * kBigThreads < held && before < k_rem; ++g) {
            const int i = group_begin(g);
            const f32x4 again = load_group(i);
            uint32_t four = 0, total;
#pragma unroll
            for (int e = 0; e < 4; ++e) four |= key_of(again[e]) == lowest ? 1u << e : 0u;
            four &= there_of(i);
            uint32_t number = before + block_excl_scan<kBigThreads>((uint32_t)__popc(four), wave_tot, &total);
#pragma unroll 1
            for (; four && number < k_rem; four &= four - 1u, ++number)
                put_tie_row(k, (uint32_t)k - k_rem + number, (uint32_t)(seg.begin + (i < last ? i : last) + __ffs((int)four) - 1), lowest, score, idx_out, val_out, s, seg.begin, seg.end);
            before += total;
        }
    }
    const int n = (int)(fill < (uint32_t)kPickCap ? fill : (uint32_t)kPickCap);
    for (int e = threadIdx.x; e < n; e += kBigThreads) {
        const uint32_t i = place[e] < (uint32_t)len ? place[e] : 0u;
        sel[slot((uint32_t)e)] = compose(key_of(seg_score[i]), (uint32_t)seg.begin + i);
    }
    if (SORT && !exact && n > k && pow2_at_least(n) > pow2_at_least(k)) {
        // what the sort may leave out: the words up to the end of rank k's bin that are not selected, whatever lies below the bin
        // included (the comparison lets every NaN in, those with the sign bit below every bound)
        for (int i = threadIdx.x; i < kBins; i += kBigThreads) hist[i] = 0;
        __syncthreads();   // (and the words are there)
        for (int e = threadIdx.x; e < n; e += kBigThreads) atomicAdd(&hist[first_digit_of((uint32_t)(sel[slot((uint32_t)e)] >> 32))], 1u);
        __syncthreads();
        find_bucket(hist, (uint32_t)k, wave_tot, found);
        uint32_t bin_lowest, bin_width;
        first_digit_range(found[0], bin_lowest, bin_width);
        lowest = 0;
        width = bin_lowest + bin_width;
        k_rem = found[1];
        exact = true;
    }
    // spare words and those behind the last must read as "below everything"
    const int n_raw = n > 0 ? (int)slot((uint32_t)n - 1u) + 1 : 0;
    for (int i = threadIdx.x; i < n_raw + 3; i += kBigThreads)
        if (i % 33 == 32 || i >= n_raw) sel[i] = 0;
    __syncthreads();
    write_collection<SORT>(sel, place, hist, &fill, &n_own, n, k, share, part, k_rem, lowest, width, exact, score, idx_out, val_out, s, seg);
}

// The largest keys of blocks (those that are asked for), for scores that nobody has held before: a workgroup to kMaximaChunk entries of
// a segment (first_block counts these).  Bound by the scores' way from memory.  The grid is segments by the longest one's chunks where
// that begins few workgroups in vain, else the chunks of all segments, each of which looks its segment up (0.3 us).  (Always the
// former began workgroups by the million where one segment is long among many: 1,000 of 1,000 and one of 4 M, k = 100, 1,762 us for
// the call, now 57; 0.4 us for a thousand of them.)
constexpr int kMaximaChunk = 4096;
constexpr int64_t kMaximaSpare = 1024;
template <class Table>
__global__ void __launch_bounds__(256) maxima_kernel(const float* __restrict__ score, Table segs, int n_seg, uint32_t* __restrict__ max16, uint32_t* __restrict__ max64,
                                                     uint32_t* __restrict__ max256)
{
    const bool by_segment = (int)gridDim.y == n_seg;
    const int s = by_segment ? (int)blockIdx.y : segment_of_block(segs.table(), n_seg, (int)blockIdx.x);
    const SegT seg = segs.at(s);
    const int64_t base = seg.begin + (int64_t)((int)blockIdx.x - (by_segment ? 0 : seg.first_block)) * kMaximaChunk + 4 * (int64_t)threadIdx.x;
    f32x4 val[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const int64_t i = base + 1024 * g;
        val[g] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (i + 4 <= seg.end) {
            val[g] = *reinterpret_cast<const f32x4_a4*>(score + i);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (i + e < seg.end) val[g][e] = score[i + e];
        }
    }
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const int64_t i = base + 1024 * g;
        uint32_t top = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t key = i + e < seg.end ? key_of(val[g][e]) : 0u;
            top = key > top ? key : top;
        }
        note_maxima<4>(top, i, kWave - 1, seg.end, s, max16, max64, max256);
    }
}

// Ties, all of the key `lowest`, in index order: the tie of rank r owns row behind + r, and k_rem of them are wanted.  A wavefront takes
// 16 x 64 neighbouring entries; one exchange of the wavefronts' counts per sweep.
__device__ __forceinline__ void write_ties(const float* __restrict__ score, const SegT& seg, uint32_t lowest, int k, uint32_t k_rem, uint32_t* wave_tot,
                                           int32_t* __restrict__ idx_out, float* __restrict__ val_out, int s)
{
    const int len = (int)(seg.end - seg.begin), lane = lane_id(), wave = threadIdx.x >> 6;
    const float* seg_score = score + seg.begin;
    const uint32_t behind = (uint32_t)k - k_rem;
    uint32_t before = 0;
    for (int row = 0; row < len && before < k_rem; row += kRow) {
        const int first = row + wave * (kWave * kBigPer) + lane;
        uint32_t before_mine[kBigPer], wave_ties = 0;
#pragma unroll
        for (int j = 0; j < kBigPer; ++j) {
            const int i = first + j * kWave;
            const bool tie = i < len && key_of(seg_score[i < len ? i : 0]) == lowest;
            const unsigned long long m = __ballot(tie);
            before_mine[j] = tie ? wave_ties + (uint32_t)__popcll(m & ((1ull << lane) - 1ull)) : 0xFFFFFFFFu;
            wave_ties += (uint32_t)__popcll(m);
        }
        __syncthreads();
        if (lane == 0) wave_tot[wave] = wave_ties;
        __syncthreads();
        uint32_t wave_before = before, all = 0;
#pragma unroll
        for (int w = 0; w < kBigThreads / kWave; ++w) {
            wave_before += w < wave ? wave_tot[w] : 0u;
            all += wave_tot[w];
        }
#pragma unroll
        for (int j = 0; j < kBigPer; ++j)
            if (before_mine[j] != 0xFFFFFFFFu && wave_before + before_mine[j] < k_rem)
                put_tie_row(k, behind + wave_before + before_mine[j], (uint32_t)(seg.begin + first + j * kWave), lowest, score, idx_out, val_out, s, seg.begin, seg.end);
        before += all;
    }
}

// Segments of up to kPickMax entries behind whoever counted the first digit: the whole segment travels to registers while the bin is looked
// up (65,536 entries, k = 1,000: 41 us for the call; 47 read in two rows by pick_kernel).  A kernel of its own, since pick_kernel's
// registers would not hold it.
template <bool SORT>
__global__ void __launch_bounds__(kBigThreads) pick_long_kernel(const float* __restrict__ score, const SegT* __restrict__ segs, int n_seg, int n_total, int k, int share,
                                                                const uint32_t* __restrict__ ghist0, int R, int32_t* __restrict__ idx_out, float* __restrict__ val_out)
{
    __shared__ __align__(16) uint64_t sel[kPickWords];
    __shared__ __align__(16) uint32_t place[kPickCap];   // indices inside the segment; later: which words this workgroup ranks
    __shared__ uint32_t hist[kBins];          // later: the ranking's counts
    __shared__ uint32_t wave_tot[16];
    __shared__ uint32_t found[3];
    __shared__ uint32_t fill, n_own, range[2];
    const int per_xcd = (n_seg * share + kXcds - 1) / kXcds, job = (int)(blockIdx.x % kXcds) * per_xcd + (int)(blockIdx.x / kXcds);
    if (job >= n_seg * share) return;
    const int s = job / share, part = job % share;
    const SegT seg = segs[s];
    const int len = (int)(seg.end - seg.begin);
    const float* seg_score = score + seg.begin;

    // Sixteen groups of four neighbours per thread.  A group that would reach past the end of the scores starts earlier; what lies
    // outside the segment is masked out below.
    constexpr int kGroups = kPickMax / (4 * kBigThreads);
    const int last = n_total - 4 - (int)seg.begin;   // (there are more than four scores in all)
    auto group_begin = [](int g) { return (g * kBigThreads + (int)threadIdx.x) * 4; };
    f32x4 val[kGroups];
#pragma unroll
    for (int g = 0; g < kGroups; ++g) {
        if (g * 4 * kBigThreads < len) {
            const int i = group_begin(g);
            val[g] = *reinterpret_cast<const f32x4_a4*>(seg_score + (i < last ? i : last));
        }
    }
    bucket_of_pass<8>(ghist0, R, n_seg, s, (uint32_t)k, hist, wave_tot, found);
    uint32_t lowest, width, k_rem = found[1], in_bin = found[2];
    first_digit_range(found[0], lowest, width);
    if (threadIdx.x == 0) fill = n_own = range[0] = range[1] = 0;
    __syncthreads();
    // More than the limit: the bin is split (the same decision in every workgroup of the segment).  (An instruction for each of a
    // thread's sixty-four entries costs 0.4 us: a key below the range is told by the difference alone, which wraps.)
    const uint32_t limit = (uint32_t)collect_limit(k);
    uint32_t largest = 0;   // of the bin's keys
    if ((uint32_t)k - k_rem + in_bin > limit) {
        uint32_t a = 0, b = 0;
#pragma unroll
        for (int g = 0; g < kGroups; ++g) {
            if (g * 4 * kBigThreads < len) {
                const int i = group_begin(g), begun = i < last ? i : last;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const uint32_t key = key_of(val[g][e]);
                    const bool in = (uint32_t)(begun + e) < (uint32_t)len && key - lowest <= width;
                    a = in && ~key > a ? ~key : a;
                    b = in && key > b ? key : b;
                }
            }
        }
        note_range(a, b, range);
        __syncthreads();
        largest = range[1];
        lowest = ~range[0];
        width = largest - lowest;
    }
#pragma unroll 1
    for (int digits = 0; digits < 3 && width != 0u && (uint32_t)k - k_rem + in_bin > limit; ++digits) {   // (a bin spans 2^22 keys at most)
        const int shift = next_shift(width);
        for (int i = threadIdx.x; i < kBins; i += kBigThreads) hist[i] = 0;
        __syncthreads();
#pragma unroll 1
        for (int row = 0; row < len; row += kRow) {
            float again[kBigPer];
            load_sweep(seg_score, row, len, again);
#pragma unroll
            for (int j = 0; j < kBigPer; ++j) {
                const uint32_t key = key_of(again[j]);
                light_hist_add(hist, (key - lowest) >> shift, sweep_index(row, j) < len && key - lowest <= width);
            }
        }
        __syncthreads();
        find_bucket(hist, k_rem, wave_tot, found);
        lowest += found[0] << shift;
        width = (1u << shift) - 1u;
        width = largest - lowest < width ? largest - lowest : width;
        k_rem = found[1];
        in_bin = found[2];
        __syncthreads();
    }
    // entries at or above `lowest` are collected; if the ties alone are too many, those above it
    const bool ties_apart = (uint32_t)k - k_rem + in_bin > limit;
    const int n = (int)(ties_apart ? (uint32_t)k - k_rem : (uint32_t)k - k_rem + in_bin);
    {
        const float t0 = threshold_of(ties_apart ? lowest + 1u : lowest);
        uint64_t mask = 0;   // bit 4 g + e: entry e of group g is not below the threshold
#pragma unroll
        for (int g = 0; g < kGroups; ++g) {
            if (g * 4 * kBigThreads < len) {
                uint32_t four = 0;
#pragma unroll
                for (int e = 3; e >= 0; --e) four = 2 * four + (val[g][e] < t0 ? 0u : 1u);
                if ((g + 1) * 4 * kBigThreads > len) {   // the segment's last groups
                    const int i = group_begin(g), begun = i < last ? i : last, left = len - i;
                    four = left <= 0 ? 0u : (four >> (i - begun)) & (left < 4 ? (1u << left) - 1u : 15u);
                }
                mask |= (uint64_t)four << (4 * g);
            }
        }
        uint32_t at = reserve(&fill, (uint32_t)__popcll(mask));
#pragma unroll 1
        for (; mask; mask &= mask - 1, ++at) {
            const int bit = __ffsll((unsigned long long)mask) - 1;
            if (at < (uint32_t)kPickCap) place[at] = (uint32_t)(group_begin(bit >> 2) + (bit & 3));
        }
    }
    // spare words and those behind the last must read as "below everything"
    const int n_raw = n > 0 ? (int)slot((uint32_t)n - 1u) + 1 : 0;
    for (int i = threadIdx.x; i < n_raw + 3; i += kBigThreads)
        if (i % 33 == 32 || i >= n_raw) sel[i] = 0;
    __syncthreads();
    if (n > 0 && fill != (uint32_t)n) {
        // The counts come from keys, the places from comparisons with a threshold: where these found more, there are NaN
        // among the scores, and the places are collected again by key.
        __syncthreads();
        if (threadIdx.x == 0) fill = 0;
        __syncthreads();
#pragma unroll 1
        for (int row = 0; row < len; row += kRow) {
            float again[kBigPer];
            load_sweep(seg_score, row, len, again);
            uint32_t mask = 0;
#pragma unroll
            for (int j = 0; j < kBigPer; ++j) {
                const uint32_t key = key_of(again[j]);
                mask |= sweep_index(row, j) < len && (ties_apart ? key > lowest : key >= lowest) ? 1u << j : 0u;
            }
            uint32_t at = reserve(&fill, (uint32_t)__popc(mask));
#pragma unroll 1
            for (; mask; mask &= mask - 1, ++at)
                if (at < (uint32_t)kPickCap) place[at] = (uint32_t)sweep_index(row, __ffs((int)mask) - 1);
        }
        __syncthreads();
    }
    for (int e = threadIdx.x; e < n; e += kBigThreads) {
        const uint32_t i = place[e] < (uint32_t)len ? place[e] : 0u;
        sel[slot((uint32_t)e)] = compose(key_of(seg_score[i]), (uint32_t)seg.begin + i);
    }
    __syncthreads();
    write_collection<SORT>(sel, place, hist, &fill, &n_own, n, k, share, part, k_rem, lowest, width, true, score, idx_out, val_out, s, seg);
    if (ties_apart && part == 0) write_ties(score, seg, lowest, k, k_rem, wave_tot, idx_out, val_out, s);
}

// The workgroups of a segment collect from its lists, and rank as pick_kernel does.
template <bool SORT>
__global__ void __launch_bounds__(kBigThreads) pick_lists_kernel(const float* __restrict__ score, const SegT* __restrict__ segs, int n_seg, int R,
                                                                 int k, int share, int span, const uint32_t* __restrict__ ghist0,
                                                                 const uint32_t* __restrict__ ghist1, const uint32_t* __restrict__ granges,
                                                                 const Stage* __restrict__ stage, int n_stages, int32_t* __restrict__ idx_out,
                                                                 float* __restrict__ val_out)
{
    __shared__ __align__(16) uint64_t sel[kPickWords];
    __shared__ __align__(16) uint32_t place[kPickCap];   // which words this workgroup ranks
    __shared__ uint32_t hist[kBins];          // later: the ranking's counts
    __shared__ uint32_t wave_tot[16];
    __shared__ uint32_t found[3];
    __shared__ uint32_t fill, n_own;
    const int per_xcd = (n_seg * share + kXcds - 1) / kXcds, job = (int)(blockIdx.x % kXcds) * per_xcd + (int)(blockIdx.x / kXcds);
    if (job >= n_seg * share) return;
    const int s = job / share, part = job % share;
    const SegT seg = segs[s];
    const int len = (int)(seg.end - seg.begin);
    const float* seg_score = score + seg.begin;
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const int b0 = seg.first_block, n_lists = (s + 1 < n_seg ? segs[s + 1].first_block : n_stages) - b0;
    uint32_t my_count = 0;   // of list `lane`
    if (lane < n_lists) my_count = reinterpret_cast<const List*>(&stage[b0 + lane])->count;
    bucket_of_pass<8>(ghist0, R, n_seg, s, (uint32_t)k, hist, wave_tot, found);
    uint32_t lowest, width, k_rem = found[1], in_bin = found[2];
    first_digit_range(found[0], lowest, width);
    if (threadIdx.x == 0) fill = n_own = 0;
    __syncthreads();
    // More than the limit: the bin is split (the same decision in every workgroup of the segment), first by the second
    // digit, which the launch before has counted.
    const uint32_t limit = (uint32_t)collect_limit(k);
    const unsigned long long overflowed = __ballot(my_count > (uint32_t)kListCap);   // (every wavefront holds all counts)
    // The spans of lists that overflowed (a stretch of good entries, as a sorted segment has it) are gone through by the whole
    // workgroup: what(row, hi, val) for each of their sweeps.
    auto through_overflowed = [&](auto&& what) {
        for (unsigned long long left = overflowed; left; left &= left - 1ull) {
            const int lo = (__ffsll(left) - 1) * span, hi = lo + span < len ? lo + span : len;
#pragma unroll 1
            for (int row = lo; row < hi; row += kRow) {
                float again[kBigPer];
                load_sweep(seg_score, row, hi, again);
                what(row, hi, again);
            }
        }
    };
    uint32_t least = 0u, largest = 0xFFFFFFFFu;   // of the bin's keys
    auto between = [&] {
        const uint32_t last_key = lowest + width < largest ? lowest + width : largest;
        lowest = lowest > least ? lowest : least;
        width = last_key - lowest;
    };
    bool second = false;
    if ((uint32_t)k - k_rem + in_bin > limit) {
        least = ~granges[(size_t)s * kBins];
        largest = granges[(size_t)s * kBins + 1];
    }
    for (int digits = 0; digits < 3 && (uint32_t)k - k_rem + in_bin > limit && width != 0u; ++digits) {   // (a bin spans 2^22 keys at most)
        const int shift = next_shift(width);
        if (!second) {
            // (its bins begin at the first bin's lowest key)
            if (least == largest) {
                between();
                break;
            }
            bucket_of_pass<1>(ghist1, 1, n_seg, s, k_rem, hist, wave_tot, found);
            second = true;
        } else {
            for (int i = threadIdx.x; i < kBins; i += kBigThreads) hist[i] = 0;
            __syncthreads();
            auto count_sweep = [&](int row, int hi, const float (&again)[kBigPer]) {
#pragma unroll
                for (int j = 0; j < kBigPer; ++j) {
                    const uint32_t key = key_of(again[j]);
                    light_hist_add(hist, (key - lowest) >> shift, sweep_index(row, j) < hi && key - lowest <= width);
                }
            };
            for (int l = wave; l < n_lists; l += kBigThreads / kWave) {
                const uint32_t cnt = (overflowed >> l) & 1ull ? 0u : (uint32_t)__builtin_amdgcn_readlane((int)my_count, l);
                const uint64_t* from = reinterpret_cast<const List*>(&stage[b0 + l])->word;
                for (uint32_t e = 0; e < cnt; e += kWave) {
                    const uint32_t key = e + lane < cnt ? (uint32_t)(from[e + lane] >> 32) : 0u;
                    light_hist_add(hist, (key - lowest) >> shift, e + lane < cnt && key - lowest <= width);
                }
            }
            through_overflowed(count_sweep);
            __syncthreads();
            find_bucket(hist, k_rem, wave_tot, found);
        }
        lowest += found[0] << shift;
        width = (1u << shift) - 1u;
        k_rem = found[1];
        in_bin = found[2];
        between();
        __syncthreads();
    }
    // entries at or above `lowest` are collected; if the ties alone are too many, those above it
    bool ties_apart = (uint32_t)k - k_rem + in_bin > limit;
    int n = (int)(ties_apart ? (uint32_t)k - k_rem : (uint32_t)k - k_rem + in_bin);
    uint64_t tie_lists = ~0ull;   // the lists whose ties are collected
    // Whole lists hold the ties as well, and lie in index order: those up to the one in which the k_rem-th tie lies are
    // ranked with the rest, at most one list's more than k.
    static_assert(kPickCap >= PRUNER_MAX_K + kListCap, "k and a list more fit");
    if (ties_apart && overflowed == 0ull) {
        for (int l = wave; l < n_lists; l += kBigThreads / kWave) {
            const uint32_t cnt = (uint32_t)__builtin_amdgcn_readlane((int)my_count, l);
            const uint64_t* from = reinterpret_cast<const List*>(&stage[b0 + l])->word;
            uint32_t ties = 0;
            for (uint32_t e = 0; e < cnt; e += kWave) ties += (uint32_t)__popcll(__ballot(e + lane < cnt && (uint32_t)(from[e + lane] >> 32) == lowest));
            if (lane == 0) hist[l] = ties;
        }
        __syncthreads();
        const uint32_t upto = wave_inclusive_sum(lane < n_lists ? hist[lane] : 0u);
        const int enough = __popcll(__ballot(upto < k_rem));   // the list of the k_rem-th tie
        n += __builtin_amdgcn_readlane((int)upto, enough);
        tie_lists = (2ull << enough) - 1ull;
        ties_apart = false;
        __syncthreads();
    }
    auto collected = [&](uint32_t key, bool with_ties) { return with_ties ? key >= lowest : key > lowest; };
    if (n > 0) {
        for (int l = wave; l < n_lists; l += kBigThreads / kWave) {
            const bool with_ties = !ties_apart && ((tie_lists >> l) & 1ull) != 0ull;
            const uint32_t cnt = (overflowed >> l) & 1ull ? 0u : (uint32_t)__builtin_amdgcn_readlane((int)my_count, l);
            const uint64_t* from = reinterpret_cast<const List*>(&stage[b0 + l])->word;
            for (uint32_t e = 0; e < cnt; e += kWave) {
                const uint64_t w = e + lane < cnt ? from[e + lane] : 0ull;
                const unsigned long long in = __ballot(e + lane < cnt && collected((uint32_t)(w >> 32), with_ties));
                if (in == 0ull) continue;
                const int leader = __ffsll(in) - 1;
                uint32_t base = 0;
                if (lane == leader) base = atomicAdd(&fill, (uint32_t)__popcll(in));
                const uint32_t at = (uint32_t)__builtin_amdgcn_readlane((int)base, leader) + (uint32_t)__popcll(in & ((1ull << lane) - 1ull));
                if (((in >> lane) & 1ull) && at < (uint32_t)n) sel[slot(at)] = w;
            }
        }
        const float t0 = threshold_of(ties_apart ? lowest + 1u : lowest);
        through_overflowed([&](int row, int hi, const float (&again)[kBigPer]) {
            uint32_t mask = 0, numbers = 0;   // not below the threshold; those of them that are numbers
#pragma unroll
            for (int j = kBigPer - 1; j >= 0; --j) {
                mask = 2 * mask + (again[j] < t0 ? 0u : 1u);
                numbers = 2 * numbers + (again[j] >= t0 ? 1u : 0u);
            }
            if (row + kRow > hi || __ballot(mask != numbers) != 0ull) {   // (an end, or NaN: the keys decide)
                mask = 0;
#pragma unroll
                for (int j = 0; j < kBigPer; ++j) mask |= sweep_index(row, j) < hi && collected(key_of(again[j]), !ties_apart) ? 1u << j : 0u;
            }
            uint32_t at = reserve(&fill, (uint32_t)__popc(mask));
            for (; mask; mask &= mask - 1, ++at) {
                const int i = (int)sweep_index(row, __ffs(mask) - 1);
                if (at < (uint32_t)n) sel[slot(at)] = compose(key_of(seg_score[i]), (uint32_t)seg.begin + (uint32_t)i);
            }
        });
    }
    __syncthreads();
    n = fill < (uint32_t)n ? (int)fill : n;   // (lists that hold their span's k best have fewer words than the counts say)
    // spare words and those behind the last must read as "below everything"
    const int n_raw = n > 0 ? (int)slot((uint32_t)n - 1u) + 1 : 0;
    for (int i = threadIdx.x; i < n_raw + 3; i += kBigThreads)
        if (i % 33 == 32 || i >= n_raw) sel[i] = 0;
    __syncthreads();
    write_collection<SORT>(sel, place, hist, &fill, &n_own, n, k, share, part, k_rem, lowest, width, true, score, idx_out, val_out, s, seg);
    if (ties_apart && part == 0) write_ties(score, seg, lowest, k, k_rem, wave_tot, idx_out, val_out, s);
}

// ---- blocks route -------------------------------------------------------------------------------------------------------
// What the levels route leaves (k above kLevelMostK, or a segment above kLevelMax) of a few long segments, at most one entry in 768: two launches, with the largest keys of 256 neighbours that
// whoever held the scores left.
//   1. kParts workgroups per segment.  Each finds, for itself, at least k blocks by (maximum, then index), at most kMostBlocks, and goes through its part of
//      them, neighbours in index order: what exceeds the bound to a list, and the indices of what equals it, in order, to another.
//      An entry of another block has the largest entries of k blocks before it.  Where a part alone has k or more above the bound (a
//      stretch of good entries), the part has a higher bound of its own.
//   2. `share` workgroups per segment collect from the lists and rank as pick_kernel does.  On scores in no particular order all
//      of the lists: of m blocks about m ln(m / (m - k)) entries reach the bound.  Where fewer than k are above it, as among the copies
//      of the explorer's later steps, the first of those that equal it; else the lists are narrowed digit by digit.
// The bound: every eighth maximum is counted (their keys' range, then digits of it) and a rank a little beyond the k-th block's
// taken; how many blocks reach that is then known exactly, and where they are too many or too few all maxima are counted.
// Bound by latencies, and by the way of the maxima (256 KB for 16.8 M entries) into each compute unit: 5.4 us of the first launch's
// 22.4 until they are there, 6.2 for the bound, 2.6 for the blocks' numbers, 2.5 until the blocks are there, 4.3 for the lists.
// 16.8 M and 4.2 M, k = 4,096: 22.4 + 15.0 us, where clearing histograms and the four launches of the spans route took 4.5 + 41; on the
// explorer's populations of copies 32.6 + 17.1 against 4.7 + 79.  From 768 entries per selected one on: 1 x 3.2 M, k = 4,096, 45 -> 39 us for
// the call, 1 x 800,000, k = 1,025, 38.5 -> 29.6; below, the bound that k blocks reach leaves too many entries (390 of them: 42 -> 49).  Sorted scores
// 5 M, k = 100, 57 -> 36; 16 M, k = 4,096, 99 -> 67.  Slower than by spans are some at this line only: 3.2 M, k = 4,096, sorted with 20,000
// good ones in the middle 50 -> 57.5, with 300 values 40 -> 47.5.  More segments: the spans route shares out the scores as well.
constexpr int kHeldQuads = 16;                                                        // of maxima, per thread
constexpr int64_t kBlocksMax = (int64_t)4 * kHeldQuads * kBigThreads * 256;           // entries of a segment
constexpr int kBlocksSegments = 4;
constexpr int64_t kBlocksSparse = 768;                                                // entries per selected one, at least: 3 k blocks (see above)
__host__ __device__ constexpr int parts_limit(int k) { return k + 3 * k / 4 + 256; }  // words that are ranked without narrowing
constexpr int kParts = kWave;                                                         // lists of a segment: a lane knows one's counts
constexpr int kPartBlocks = 6 * (kBigThreads / kWave);                                // blocks of a part
constexpr int kMostBlocks = kParts * kPartBlocks;
static_assert(kMostBlocks >= PRUNER_MAX_K, "the k best blocks fit");

static_assert(kPickCap >= parts_limit(PRUNER_MAX_K), "a collection fits");

constexpr int kPartWords = collect_limit(PRUNER_MAX_K);   // (room for little more than k: for k alone a bound of a part's own takes every digit)
struct PartList {
    uint32_t above, ties, bound, top;     // top: the part's largest key
    uint64_t word[kPartWords];            // of entries above `bound`
    uint32_t tie[PRUNER_MAX_K];           // indices, in order, of entries that equal it
};

// A thread's part of `four` counts per row (rows in order, the lanes' order in each), wavefront after wavefront: calls
// put(row, first number) with the number of things before this thread's of that row.  All threads; returns the total.
template <int ROWS, class Count, class Put>
__device__ __forceinline__ uint32_t number_rows(uint32_t* wave_tot, Count&& count, Put&& put)
{
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    uint32_t before[ROWS], sum = 0;
#pragma unroll
    for (int j = 0; j < ROWS; ++j) {
        const uint32_t mine = count(j), upto = wave_inclusive_sum(mine);
        before[j] = sum + upto - mine;
        sum += (uint32_t)__builtin_amdgcn_readlane((int)upto, kWave - 1);
    }
    __syncthreads();   // (wave_tot may still be read)
    if (lane == 0) wave_tot[wave] = sum;
    __syncthreads();
    uint32_t total = 0, wave_before = 0;
#pragma unroll
    for (int w = 0; w < kBigThreads / kWave; ++w) {
        wave_before += w < wave ? wave_tot[w] : 0u;
        total += wave_tot[w];
    }
#pragma unroll
    for (int j = 0; j < ROWS; ++j) put(j, wave_before + before[j]);
    return total;
}

// The sum of all threads' values.
__device__ __forceinline__ uint32_t sum_of_all(uint32_t mine, uint32_t* wave_tot)
{
    const uint32_t upto = wave_inclusive_sum(mine);
    __syncthreads();
    if (lane_id() == kWave - 1) wave_tot[threadIdx.x >> 6] = upto;
    __syncthreads();
    uint32_t total = 0;
#pragma unroll
    for (int w = 0; w < kBigThreads / kWave; ++w) total += wave_tot[w];
    return total;
}

template <class Table>
__global__ void __launch_bounds__(kBigThreads) block_lists_kernel(const float* __restrict__ score, Table segs, int n_total, int k, const uint32_t* __restrict__ max256,
                                                                  PartList* __restrict__ lists)
{
    __shared__ __attribute__((aligned(16))) uint8_t nibble[kBigThreads * kHeldQuads];
    __shared__ uint32_t hist[kBins], blocks[kMostBlocks], wave_tot[16], found[3], range[2], fill, top;
    const int s = blockIdx.x / kParts, part = blockIdx.x % kParts, lane = lane_id(), wave = threadIdx.x >> 6;
    const SegT seg = segs.at(s);
    const int len = (int)(seg.end - seg.begin), n256 = (len + 255) >> 8, n_quads = (n256 + 3) >> 2;
    const float* const seg_score = score + seg.begin;
    const uint32_t* const maxima = max256 + block_max_slot(seg.begin, s);

    // the maxima, `rows` rows of 64 quads per wavefront, neighbours
    const int rows = (n_quads + kBigThreads - 1) / kBigThreads;   // at most kHeldQuads
    auto quad = [&](int j) -> int { return (wave * rows + j) * kWave + lane; };
    u32x4 v[kHeldQuads];
#pragma unroll
    for (int j = 0; j < kHeldQuads; ++j) {
        v[j] = u32x4{0u, 0u, 0u, 0u};
        if (j < rows && quad(j) < n_quads) v[j] = maxima_at(maxima, 4 * quad(j), n256);
    }
    if (threadIdx.x < 2) range[threadIdx.x] = 0;
    if (threadIdx.x == 2) fill = top = 0;
    __syncthreads();
    // blocks whose maximum is at or above `key` (above zero), four bits a row; in 0 no block past the last
    uint32_t mask[2];
    auto reach = [&](uint32_t key) {
        constexpr int kHalf = kHeldQuads / 2;
        static_assert(kHeldQuads == 16, "two words of masks");
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            mask[h] = 0;
#pragma unroll
            for (int i = 4 * kHalf - 1; i >= 0; --i) mask[h] = 2 * mask[h] + (v[h * kHalf + (i >> 2)][i & 3] >= key ? 1u : 0u);
        }
        return sum_of_all((uint32_t)(__popc(mask[0]) + __popc(mask[1])), wave_tot);
    };
    // The bound: a digit at a time of the first maxima of every other row's quads; where what they show leaves too few or too many, of all.
    // (A maximum of 0, which names a NaN, is not counted: a bound of 0 serves.)
    uint32_t bound = 0, n_reach = 0, n_above = 0;
#pragma unroll 1
    for (int attempt = 0; attempt < 2; ++attempt) {
        uint32_t n_mine = 0, lowest = 1u, width = ~0u - 1u;
        if (attempt == 0) {
            uint32_t not_least = 0, most = 0;
#pragma unroll
            for (int j = 0; j < kHeldQuads; j += 2) {
                const uint32_t x = v[j][0];
                most = x > most ? x : most;
                not_least = x != 0u && ~x > not_least ? ~x : not_least;
                n_mine += x != 0u ? 1u : 0u;
            }
            note_range(not_least, most, range);
        } else {
#pragma unroll
            for (int j = 0; j < kHeldQuads; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) n_mine += v[j][e] != 0u ? 1u : 0u;
        }
        const uint32_t n_counted = sum_of_all(n_mine, wave_tot);   // (a barrier: the range is there)
        uint32_t rank = (uint32_t)k, spare = (uint32_t)(kMostBlocks - k);
        if (attempt == 0) {
            const float expected = (float)k * (float)n_counted / (float)n256;
            rank = (uint32_t)(expected + 4.f * __builtin_sqrtf(expected)) + 1u;
            rank = rank < n_counted ? rank : n_counted;
            spare = rank / 8;
            lowest = ~range[0];
            width = range[1] - lowest;
        }
        if (rank == 0u || n_counted < rank) {
            lowest = 0u;
            width = 0u;
        }
#pragma unroll 1
        while (width != 0u) {
            const int shift = next_shift(width);
            for (int i = threadIdx.x; i < kBins; i += kBigThreads) hist[i] = 0;
            __syncthreads();
            if (attempt == 0) {
#pragma unroll
                for (int j = 0; j < kHeldQuads; j += 2)
                    if (j < rows) light_hist_add(hist, (v[j][0] - lowest) >> shift, v[j][0] >= lowest && v[j][0] - lowest <= width);
            } else {
#pragma unroll 1
                for (int i = threadIdx.x; i < rows * kBigThreads; i += kBigThreads) {
                    const u32x4 w = maxima_at(maxima, 4 * (i < n_quads ? i : 0), n256);
#pragma unroll
                    for (int e = 0; e < 4; ++e) light_hist_add(hist, (w[e] - lowest) >> shift, i < n_quads && w[e] >= lowest && w[e] - lowest <= width);
                }
            }
            __syncthreads();
            find_bucket(hist, rank, wave_tot, found);
            lowest += found[0] << shift;
            width = (1u << shift) - 1u;
            rank = found[1];
            if (found[2] - rank <= spare) break;
        }
        bound = lowest;
        n_reach = reach(bound);
        if (n_reach >= (uint32_t)k && n_reach <= (uint32_t)kMostBlocks) break;
        if (n_reach < (uint32_t)k) continue;
        n_above = bound == ~0u ? 0u : reach(bound + 1u);
        if (n_above <= (uint32_t)kMostBlocks) break;
    }
    // all that reach the bound; if they are too many, those above it, and if these are fewer than k, the first that equal it
    const bool ties_apart = n_reach > (uint32_t)kMostBlocks;
    const uint32_t n_ties = ties_apart && n_above < (uint32_t)k ? (uint32_t)k - n_above : 0u;
    // A thread's maxima lie row by row; their bits go to the thread that numbers 64 neighbours, through LDS.
    auto in_order = [&](const uint32_t(&m)[2]) {
        uint8_t* const mine = nibble + wave * (kHeldQuads * kWave);
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kHeldQuads; ++j) mine[j * kWave + lane] = (uint8_t)((m[j / 8] >> (4 * (j % 8))) & 15u);
        __syncthreads();
        static_assert(kHeldQuads == 16, "sixteen nibbles of a row per lane");
        const u32x4 sixteen = reinterpret_cast<const u32x4*>(mine)[lane];
        uint64_t bits = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            uint32_t x = sixteen[e];
            x = (x | x >> 4) & 0x00FF00FFu;
            bits |= (uint64_t)((x | x >> 8) & 0xFFFFu) << (16 * e);
        }
        return (lane >> 2) < rows ? bits : 0ull;
    };
    uint32_t total;
    uint64_t chosen;
    if (n_ties != 0u) {
        const uint32_t over[2] = {bound == ~0u ? 0u : mask[0], bound == ~0u ? 0u : mask[1]};   // above it
        reach(bound);
        const uint32_t level[2] = {mask[0] & ~over[0], mask[1] & ~over[1]};
        chosen = in_order(over);
        uint64_t equal = in_order(level);
        uint32_t number = block_excl_scan<kBigThreads>((uint32_t)__popcll(equal), wave_tot, &total);
        if (number + (uint32_t)__popcll(equal) <= n_ties) {
            chosen |= equal;
        } else {
#pragma unroll 1
            for (; equal && number < n_ties; equal &= equal - 1ull, ++number) chosen |= equal & (0ull - equal);
        }
    } else {
        chosen = in_order(mask);
    }
    uint32_t number = block_excl_scan<kBigThreads>((uint32_t)__popcll(chosen), wave_tot, &total);
    const uint32_t n_blocks = total;
#pragma unroll 1
    for (; chosen; chosen &= chosen - 1ull, ++number)
        if (number < (uint32_t)kMostBlocks) blocks[number] = (uint32_t)(256 * wave * rows + 64 * lane + __ffsll((unsigned long long)chosen) - 1);
    if (ties_apart && n_ties == 0u) bound += 1u;   // (k blocks are above it)
    __syncthreads();

    // this part's blocks, six to a wavefront
    constexpr int kPer = kPartBlocks / (kBigThreads / kWave);
    const int nb = (int)(n_blocks < (uint32_t)kMostBlocks ? n_blocks : (uint32_t)kMostBlocks), b_lo = part * nb / kParts, b_hi = (part + 1) * nb / kParts;
    const int last = n_total - 4 - (int)seg.begin;   // (the segment is long: at least 0 or a negative number whose entry exists)
    int at[kPer];
    f32x4 val[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int b = b_lo + wave * kPer + j;
        at[j] = b < b_hi ? 256 * (int)blocks[b] + 4 * lane : len;
        val[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (at[j] < len) val[j] = *reinterpret_cast<const f32x4_a4*>(seg_score + (at[j] < last ? at[j] : last));
    }
    uint32_t key[kPer][4], live[kPer];   // live: the entries that reach the bound; the others' keys are 0
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int begun = at[j] < last ? at[j] : last;
        live[j] = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t x = key_of(val[j][e]);
            const bool in = at[j] < len && begun + e >= at[j] && begun + e < len && x >= bound;
            key[j][e] = in ? x : 0u;
            live[j] |= in ? 1u << e : 0u;
        }
        at[j] = begun;
    }
    auto count = [&](auto&& what) {
        uint32_t n = 0;
#pragma unroll
        for (int j = 0; j < kPer; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) n += what(key[j][e]) ? 1u : 0u;
        return n;
    };
    uint32_t most = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) most = key[j][e] > most ? key[j][e] : most;
    most = wave_inclusive_max(most);
    if (lane == kWave - 1 && most) atomicMax(&top, most);
    uint32_t n_list = sum_of_all(count([&](uint32_t x) { return x > bound; }), wave_tot);
    bool with_ties = n_list < (uint32_t)k;
    if (!with_ties) {
        // a bound of its own, which k of this part's entries reach and little more than k
        const uint32_t enough = (uint32_t)collect_limit(k);
        uint32_t lowest = bound + 1u, width = top - lowest, rank = (uint32_t)k, reach = n_list;
#pragma unroll 1
        while (reach > enough && width != 0u) {
            const int shift = next_shift(width);
            __syncthreads();
            for (int i = threadIdx.x; i < kBins; i += kBigThreads) hist[i] = 0;
            __syncthreads();
#pragma unroll
            for (int j = 0; j < kPer; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) light_hist_add(hist, (key[j][e] - lowest) >> shift, key[j][e] >= lowest && key[j][e] - lowest <= width);
            __syncthreads();
            find_bucket(hist, rank, wave_tot, found);
            lowest += found[0] << shift;
            width = (1u << shift) - 1u;
            rank = found[1];
            reach = (uint32_t)k - rank + found[2];
        }
        with_ties = reach > enough;   // (one value: fewer than k are above it)
        bound = with_ties ? lowest : lowest - 1u;
        n_list = sum_of_all(count([&](uint32_t x) { return x > bound; }), wave_tot);
    }
    PartList& mine = lists[blockIdx.x];
    uint32_t to = reserve(&fill, count([&](uint32_t x) { return x > bound; }));
    uint32_t equal[kPer], any = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        equal[j] = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (key[j][e] > bound) {
                if (to < (uint32_t)kPartWords) mine.word[to] = compose(key[j][e], (uint32_t)seg.begin + (uint32_t)(at[j] + e));
                ++to;
            }
            equal[j] |= with_ties && ((live[j] >> e) & 1u) && key[j][e] == bound ? 1u << e : 0u;
        }
        any |= equal[j];
    }
    uint32_t n_equal = 0;
    if (__syncthreads_or((int)any)) {
        n_equal = number_rows<kPer>(wave_tot, [&](int j) { return (uint32_t)__popc(equal[j]); }, [&](int j, uint32_t number) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if ((equal[j] >> e) & 1u) {
                    if (number < (uint32_t)k) mine.tie[number] = (uint32_t)seg.begin + (uint32_t)(at[j] + e);
                    ++number;
                }
        });
    }
    if (threadIdx.x == 0) {
        mine.above = n_list;
        mine.ties = n_equal < (uint32_t)k ? n_equal : (uint32_t)k;
        mine.bound = bound;
        mine.top = top;
    }
}

template <bool SORT, class Table>
__global__ void __launch_bounds__(kBigThreads) pick_parts_kernel(const float* __restrict__ score, Table segs, int n_seg, int k, int share, const PartList* __restrict__ lists,
                                                                 int32_t* __restrict__ idx_out, float* __restrict__ val_out)
{
    __shared__ __align__(16) uint64_t sel[kPickWords];
    __shared__ __align__(16) uint32_t place[kPickCap];   // which words this workgroup ranks
    __shared__ uint32_t hist[kBins];                     // later: the ranking's counts
    __shared__ uint32_t wave_tot[16], found[3], fill, n_own, range[2], above_upto[kParts], ties_upto[kParts], bound_of[kParts];
    const int per_xcd = (n_seg * share + kXcds - 1) / kXcds, job = (int)(blockIdx.x % kXcds) * per_xcd + (int)(blockIdx.x / kXcds);
    if (job >= n_seg * share) return;
    const int s = job / share, part = job % share, lane = lane_id(), wave = threadIdx.x >> 6;
    const SegT seg = segs.at(s);
    const PartList* const own_lists = lists + (size_t)s * kParts;
    constexpr int kMine = kParts / (kBigThreads / kWave);   // lists of a wavefront
    constexpr int kAhead = 2;                               // words of each that are asked for at once, per lane (the lists hold kPartWords: inside)
    uint64_t ahead[kMine][kAhead];
#pragma unroll
    for (int q = 0; q < kMine; ++q)
#pragma unroll
        for (int a = 0; a < kAhead; ++a) ahead[q][a] = own_lists[wave * kMine + q].word[a * kWave + lane];
    uint32_t my_above = own_lists[lane].above, my_ties = own_lists[lane].ties;
    const uint32_t my_bound = own_lists[lane].bound, my_top = own_lists[lane].top;
    if (threadIdx.x == 0) fill = n_own = range[0] = range[1] = 0;
    __syncthreads();
    // what a list of k or more shows: the others' entries below its bound are none of the k best
    const uint32_t shown = (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_max(my_above + my_ties >= (uint32_t)k ? my_bound + (my_above >= (uint32_t)k ? 1u : 0u) : 0u), kWave - 1);
    if (my_top < shown) my_above = my_ties = 0;
    const uint32_t upto_above = wave_inclusive_sum(my_above), upto_ties = wave_inclusive_sum(my_ties);
    const uint32_t n_above = (uint32_t)__builtin_amdgcn_readlane((int)upto_above, kWave - 1), n_ties = (uint32_t)__builtin_amdgcn_readlane((int)upto_ties, kWave - 1);
    const bool one_bound = __ballot(my_bound != (uint32_t)__builtin_amdgcn_readfirstlane((int)my_bound)) == 0ull;
    const uint32_t limit = (uint32_t)parts_limit(k);
    const uint32_t n_listed = n_above + n_ties;
    uint32_t n = n_listed;
    const bool whole = n <= limit, first_ties = !whole && one_bound && n_above < (uint32_t)k;
    if (threadIdx.x < kParts) {
        above_upto[threadIdx.x] = upto_above;
        ties_upto[threadIdx.x] = upto_ties;
        bound_of[threadIdx.x] = my_bound;
    }
    __syncthreads();
    auto of_list = [&](uint32_t mine, int l) { return (uint32_t)__builtin_amdgcn_readlane((int)mine, l); };
    // the list that number t of the lists' words (or ties), one list after the other, lies in: how many end at or before t
    auto list_of = [&](const uint32_t* upto, uint32_t t) {
        int l = 0;
#pragma unroll
        for (int step = kParts / 2; step > 0; step >>= 1) l += upto[l + step - 1] <= t ? step : 0;
        return l;
    };
    constexpr int kWords = kPickCap / kBigThreads;   // of a thread at a time
    if (__builtin_expect(whole || first_ties, 1)) {   // (nearly always)
        // all entries above the bound, and the ties, or the first of them: every word's place is known
        const uint32_t take = whole ? n_ties : (uint32_t)k - n_above;
        n = n_above + take;
        // (a tie's list by bisection: all of a thread's are under way at once, however long the lists are)
        uint32_t from[kWords], tie_key[kWords];
#pragma unroll
        for (int i = 0; i < kWords; ++i) {
            const uint32_t t = (uint32_t)(i * kBigThreads) + threadIdx.x;
            from[i] = tie_key[i] = 0;
            if (t < take) {
                const int l = list_of(ties_upto, t);
                from[i] = own_lists[l].tie[t - (l > 0 ? ties_upto[l - 1] : 0u)];
                tie_key[i] = bound_of[l];
            }
        }
#pragma unroll
        for (int q = 0; q < kMine; ++q) {
            const int l = wave * kMine + q;
            const uint32_t above = of_list(my_above, l), before = of_list(upto_above, l) - above;
#pragma unroll
            for (int a = 0; a < kAhead; ++a)
                if (a * kWave + lane < (int)above) sel[slot(before + a * kWave + lane)] = ahead[q][a];
        }
#pragma unroll 1
        for (unsigned long long left = __ballot(my_above > (uint32_t)(kAhead * kWave)); left; left &= left - 1ull) {
            const int l = __ffsll(left) - 1;
            const uint32_t above = of_list(my_above, l), before = of_list(upto_above, l) - above;
            for (uint32_t e = kAhead * kWave + threadIdx.x; e < above; e += kBigThreads) sel[slot(before + e)] = own_lists[l].word[e];
        }
#pragma unroll
        for (int i = 0; i < kWords; ++i) {
            const uint32_t t = (uint32_t)(i * kBigThreads) + threadIdx.x;
            if (t < take) sel[slot(n_above + t)] = compose(tie_key[i], from[i]);
        }
    } else {
        // What reaches what is shown is gathered, a thread's words of kPickCap under way at once (list after list, 1,024 words at a time, a
        // pass over full lists took 50 us).  Where that is too much it is narrowed by the keys' digits, then, where one key remains, by its
        // entries' indices: words at or above `least`.
        uint64_t least = (uint64_t)shown << 32;
        bool held = false;   // sel holds the words that are looked at; else the lists do
        uint32_t n_words = n_listed;
        auto word_at = [&](uint32_t t) -> uint64_t {
            if (t >= n_words) return 0ull;
            if (held) return sel[slot(t)];
            const bool above = t < n_above;
            const uint32_t* const upto = above ? above_upto : ties_upto;
            const uint32_t number = above ? t : t - n_above;
            const int l = list_of(upto, number);
            const uint32_t at = number - (l > 0 ? upto[l - 1] : 0u);
            return above ? own_lists[l].word[at] : compose(bound_of[l], own_lists[l].tie[at]);
        };
#pragma unroll 1
        for (int round = 0;; ++round) {
#pragma unroll 1
            for (uint32_t base = 0; base < n_words; base += (uint32_t)kPickCap) {
                uint64_t word[kWords];
                uint32_t in = 0;
#pragma unroll
                for (int i = 0; i < kWords; ++i) word[i] = word_at(base + (uint32_t)(i * kBigThreads) + threadIdx.x);
#pragma unroll
                for (int i = 0; i < kWords; ++i) in |= word[i] != 0ull && word[i] >= least ? 1u << i : 0u;
                if (held) __syncthreads();   // (at most kPickCap: all have been read)
                uint32_t to = reserve(&fill, (uint32_t)__popc(in));
#pragma unroll
                for (int i = 0; i < kWords; ++i) {
                    if (!((in >> i) & 1u)) continue;
                    if (to < (uint32_t)kPickCap) sel[slot(to)] = word[i];
                    ++to;
                }
            }
            __syncthreads();
            n = fill;
            if (n <= limit) break;   // (after the second round always)
            __syncthreads();
            if (threadIdx.x == 0) fill = 0;
            held = n <= (uint32_t)kPickCap;
            if (held) n_words = n;
            // every word: what(whether there is one, word), the lanes of a wavefront together
            auto each = [&](auto&& what) {
#pragma unroll 1
                for (uint32_t t = 0; t < n_words; t += kBigThreads) {
                    const uint64_t w = word_at(t + threadIdx.x);
                    what(w != 0ull, w);
                }
            };
            uint32_t not_least = 0, most = 0;
            each([&](bool there, uint64_t w) {
                const uint32_t key = (uint32_t)(w >> 32);
                most = there && key > most ? key : most;
                not_least = there && ~key > not_least ? ~key : not_least;
            });
            note_range(not_least, most, range);
            __syncthreads();
            uint32_t lowest = ~range[0] > shown ? ~range[0] : shown, width = range[1] - lowest, rank = (uint32_t)k, index_lowest = 0;
            bool by_key = true;
            if (width == 0u) by_key = false, index_lowest = 0xFFFFFFFFu - (uint32_t)(seg.end - 1), width = (uint32_t)(seg.end - seg.begin) - 1u;
#pragma unroll 1
            for (;;) {
                const int shift = next_shift(width);
                const uint32_t base = by_key ? lowest : index_lowest;
                for (int i = threadIdx.x; i < kBins; i += kBigThreads) hist[i] = 0;
                __syncthreads();
                each([&](bool there, uint64_t w) {
                    const uint32_t x = by_key ? (uint32_t)(w >> 32) : (uint32_t)w;
                    light_hist_add(hist, (x - base) >> shift, there && (by_key || (uint32_t)(w >> 32) == lowest) && x >= base && x - base <= width);
                });
                __syncthreads();
                find_bucket(hist, rank, wave_tot, found);
                (by_key ? lowest : index_lowest) += found[0] << shift;
                width = (1u << shift) - 1u;
                rank = found[1];
                if ((uint32_t)k - rank + found[2] <= limit) break;
                if (width == 0u) {   // (an index is one entry's: this was a key)
                    by_key = false;
                    index_lowest = 0xFFFFFFFFu - (uint32_t)(seg.end - 1);
                    width = (uint32_t)(seg.end - seg.begin) - 1u;
                }
            }
            least = ((uint64_t)lowest << 32) | index_lowest;
        }
    }
    // spare words and those behind the last must read as "below everything"
    const int n_raw = n > 0 ? (int)slot(n - 1u) + 1 : 0;
    for (int i = threadIdx.x; i < n_raw + 3; i += kBigThreads)
        if (i % 33 == 32 || i >= n_raw) sel[i] = 0;
    __syncthreads();
    write_collection<SORT>(sel, place, hist, &fill, &n_own, (int)n, k, share, part, (uint32_t)k, 0u, ~0u, false, score, idx_out, val_out, s, seg, whole || first_ties);
}

struct Layout {
    size_t segs, state, hist, stage, max256, max64, max16, parts, with_parts, total;
    size_t stage_slots;
    int R;
};

constexpr int kFewSegs = 64;   // segment tables up to this length are built on the stack
constexpr int kComputeUnits = 256;   // of the part this library is written for (gfx950 in its full configuration)

int hist_copies(int32_t n_sg) { return n_sg <= 16 ? 8 : n_sg <= 64 ? 4 : 1; }

// entries per workgroup of the spans and lists routes: whole sweeps, and at most 512 workgroups per launch, which is what 256
// CUs hold at once (two workgroups of 1024 threads each): a launch then runs as a single wave of workgroups
// (quarter sweeps for populations that leave CUs idle were measured: more workgroups add to the segment's histograms
// and lists, 11 -> 14 us for the funnel launch on a million entries)
int64_t span_for(int64_t n, int32_t n_sg)
{
    const int64_t sweeps = (n + kRow - 1) / kRow + n_sg;
    return kRow * ((sweeps + 511) / 512);
}

// with_block_max: room for the largest key of every 16, 64 and 256 entries (the one part that grows with n, 21 bytes per 64 entries).
// A call has histograms and staged entries, or the finer maxima, or the lists of parts: they lie in the same place, and no call
// needs more than it did with the digits alone, up to some 17 million entries.
// total: what a call cannot do without; with_parts: what it takes for the blocks route as well, for as many of the segments as that
// route serves, so that room for more segments serves fewer of them by the same route.
Layout layout(int64_t n, int32_t n_sg, int32_t k, bool with_block_max)
{
    (void)k;   // (what serves one k serves any)
    Layout L;
    L.R = hist_copies(n_sg);
    // workgroups of a sweep launch: at most 512 whole spans plus one partial span per segment
    const size_t sweeps = (size_t)(n / kRow);
    const size_t blocks = (sweeps < 512 ? sweeps : 512) + (size_t)n_sg + 1;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off += round_up(bytes, 256);
        return at;
    };
    L.segs = take((size_t)n_sg * sizeof(SegT));
    L.state = take((size_t)3 * n_sg * sizeof(SelState));
    // (three words more: the maxima are read in fours)
    L.max256 = with_block_max ? take(((size_t)(n >> 8) + (size_t)n_sg + 4) * sizeof(uint32_t)) : 0;
    const size_t shared = off;
    L.hist = take(((size_t)L.R + 2) * n_sg * kBins * sizeof(uint32_t));   // first digit in R copies, one each for the others
    L.stage = take(blocks * sizeof(Stage));
    L.stage_slots = blocks;
    L.total = off;
    off = shared;
    L.max64 = with_block_max ? take(((size_t)(n >> 6) + (size_t)n_sg + 4) * sizeof(uint32_t)) : 0;
    L.max16 = with_block_max ? take(((size_t)(n >> 4) + (size_t)n_sg + 4) * sizeof(uint32_t)) : 0;
    L.total = off > L.total ? off : L.total;
    off = shared;
    L.parts = with_block_max && n >= kBlocksSparse * (kLevelMostK + 1) ? take((size_t)(n_sg < kBlocksSegments ? n_sg : kBlocksSegments) * kParts * sizeof(PartList)) : shared;
    L.with_parts = off > L.total ? off : L.total;
    return L;
}

}  // namespace

size_t topk_workspace_bytes(int64_t n, int32_t n_sg, int32_t k, bool parts)
{
    if (n < 0) n = 0;
    if (n_sg < 1) n_sg = 1;
    if (k < 1) k = 1;
    const Layout L = layout(n, n_sg, k, true);
    return parts ? L.with_parts : L.total;
}


// what every selection call refuses about its segments and k (host pointers only); *longest, *shortest: of the segments
static int topk_check(const int64_t* seg_off, int32_t n_sg, int32_t k, int64_t* longest, int64_t* shortest = nullptr)
{
    if (!seg_off || n_sg < 1 || n_sg > PRUNER_MAX_SUBGRAPHS || k < 1 || k > PRUNER_MAX_K) return PRUNER_EINVAL;
    if (seg_off[0] != 0) return PRUNER_EINVAL;
    *longest = 0;
    for (int32_t s = 0; s < n_sg; ++s) {
        const int64_t len = seg_off[s + 1] - seg_off[s];
        if (len < k) return PRUNER_EINVAL;
        *longest = len > *longest ? len : *longest;
        if (shortest) *shortest = s == 0 || len < *shortest ? len : *shortest;
    }
    if (seg_off[n_sg] > 0x7FFFFFFFll) return PRUNER_EINVAL;  // indices are int32
    return PRUNER_OK;
}

int topk_prepare(const int64_t* seg_off, int32_t n_sg, int32_t k, void* workspace, size_t workspace_bytes, hipStream_t st, TopkCtx* ctx,
                 Upload* defer, bool with_block_max, bool copies)
{
    int64_t longest = 0, shortest = 0;
    const int bad = topk_check(seg_off, n_sg, k, &longest, &shortest);
    if (bad) return bad;
    const int64_t n = seg_off[n_sg];
    if (!workspace || !aligned(workspace, 256)) return PRUNER_EWORKSPACE;
    const Layout L = layout(n, n_sg, k, with_block_max);
    if (workspace_bytes < L.total) return PRUNER_EWORKSPACE;

    char* ws = static_cast<char*>(workspace);
    SegT* d_segs = reinterpret_cast<SegT*>(ws + L.segs);
    // the ranking of a segment's k rows is shared out over up to k / 32 workgroups, as long as the launch is one
    // workgroup per compute unit at most (a compute unit holds one of these workgroups at a time: a launch of more
    // takes a second round, which costs more than longer rankings do)
    int share = (k + 31) / 32;
    if (share > kComputeUnits / n_sg) share = kComputeUnits / n_sg;
    if (share < 1) share = 1;
    const bool sort = (k + 64 * share - 1) / (64 * share) * k > kSortFactor * pow2_at_least(k);   // (a collection is k words and a little more)
    // (without room for maxima: as for a large k.)  Where the draft kernel counts first digits on the way, segments held whole are the
    // better ones with fewer than two blocks of sixteen per selected entry, of which the bound leaves too many entries (the filter of
    // 6 x 16,500, k = 700: 20.3 us by digits, 27.6 by levels; of 20,000 20.4 and 20.0; 20 x 20,000 23.8 and 30.1, 25,000 24.6 and 23.2),
    // and where few workgroups share a ranking and sort (100 x 25,000, k = 512: 45.6 and 49.0, k = 256 37.7 and 35.5; 100 x 40,000 of
    // convolutions, k = 512, 67.5 and 74.5).
    const bool tiny = longest <= kTinyMax && k <= kTinyK;
    const bool better_held = defer && longest <= kPickMax && (longest < 32 * (int64_t)k || sort);
    const bool levels = with_block_max && !tiny && !better_held && longest > (defer ? kRow : kCountMax) && k <= kLevelMostK && longest <= kLevelMax;
    const bool pick = !tiny && !levels && longest <= kPickMax;
    const bool blocks_route = with_block_max && !tiny && !levels && !pick && n_sg <= kBlocksSegments && longest <= kBlocksMax && shortest >= kBlocksSparse * (int64_t)k && workspace_bytes >= L.with_parts;
    // Segments of up to two rows are counted where they are held as cheaply as by a launch of its own (20 of 30,000, k = 4,096: 44 us
    // either way), unless the draft kernel does it.
    const bool counted = pick && longest > (defer ? kRow : kCountMax);
    const int64_t span = levels || blocks_route ? kMaximaChunk : span_for(n, n_sg);   // (of the first launch that goes through the scores)

    // the segment table: on the stack when it is short (a call that must not allocate stays off the heap as well)
    SegT few[kFewSegs];
    std::vector<SegT> many;
    if (n_sg > kFewSegs) many.resize(n_sg);
    SegT* const segs = n_sg > kFewSegs ? many.data() : few;
    int64_t blocks = 0;
    for (int32_t s = 0; s < n_sg; ++s) {
        segs[s] = SegT{seg_off[s], seg_off[s + 1], (int32_t)blocks, 0};
        blocks += (seg_off[s + 1] - seg_off[s] + span - 1) / span;
    }
    // (a population of copies, as the explorer loop keeps it, would have its lists overflow as a rule: it takes the spans route)
    const bool lists = !tiny && !pick && !levels && !blocks_route && longest <= kListsMax && !copies;
    ctx->tiny = tiny;
    ctx->pick = pick;
    ctx->levels = levels;
    ctx->blocks_route = blocks_route;
    ctx->lists = lists;
    ctx->digits = !tiny && !levels && !blocks_route && (!pick || counted);
    ctx->longest = longest;
    ctx->share = share;
    ctx->sort = sort;
    ctx->n_sg = n_sg;
    ctx->k = k;
    ctx->n = n;
    ctx->span = span;
    ctx->blocks = (int32_t)blocks;
    ctx->copies = L.R;
    ctx->d_segs = d_segs;
    ctx->d_state = ws + L.state;
    ctx->d_hist = reinterpret_cast<uint32_t*>(ws + L.hist);
    ctx->d_stage = ws + L.stage;
    ctx->d_parts = ws + L.parts;
    // Block maxima pay where nearly every block of 256 entries can be stepped over: at most one entry in 1024 selected
    // in the longest segment (with k = 512 of 50,000 nine blocks in ten hold a selected entry and the maxima are one
    // more read: 10.7 -> 11.5 us measured).
    const bool sparse = ctx->digits && !pick && !lists && longest >= (int64_t)k * 1024;
    ctx->d_max16 = levels ? reinterpret_cast<uint32_t*>(ws + L.max16) : nullptr;
    ctx->d_max64 = levels && longest > 16 * (int64_t)kDirectBlocks ? reinterpret_cast<uint32_t*>(ws + L.max64) : nullptr;
    ctx->d_max256 = with_block_max && (sparse || blocks_route || (levels && longest > 64 * (int64_t)kDirectBlocks)) ? reinterpret_cast<uint32_t*>(ws + L.max256) : nullptr;
    ctx->inline_ok = false;
    static_assert(sizeof(InlineSegs) <= sizeof(ctx->inline_segs), "inline segment table");
    if (!ctx->digits) {
        if (n_sg <= kInlineSegs) {
            memset(ctx->inline_segs, 0, sizeof(InlineSegs));
            memcpy(ctx->inline_segs, segs, (size_t)n_sg * sizeof(SegT));
            ctx->inline_ok = true;
            return PRUNER_OK;
        }
        if (defer) {
            defer->bytes.assign(reinterpret_cast<const char*>(segs), reinterpret_cast<const char*>(segs + n_sg));
            defer->dst = d_segs;
            return PRUNER_OK;
        }
        return put_table(d_segs, segs, (size_t)n_sg * sizeof(SegT), st);
    }
    if ((size_t)blocks > L.stage_slots) return PRUNER_EWORKSPACE;   // cannot happen: spans are sized for at most that many
    // segment table, and histograms cleared, in one launch
    const size_t per_pass = (size_t)n_sg * kBins;
    const size_t hist_bytes = ((size_t)L.R + (pick ? 0 : 2)) * per_pass * sizeof(uint32_t);
    if (defer) {
        defer->bytes.assign(reinterpret_cast<const char*>(segs), reinterpret_cast<const char*>(segs + n_sg));
        defer->dst = d_segs;
        defer->zero = ctx->d_hist;
        defer->zero_bytes = hist_bytes;
        return PRUNER_OK;
    }
    return put_table(d_segs, segs, (size_t)n_sg * sizeof(SegT), st, ctx->d_hist, hist_bytes);
}

int topk_finish(const TopkCtx& ctx, const float* score, const int64_t* seg_off, int32_t* idx_out, float* val_out, bool noted,
                hipStream_t st)
{
    if (!score || !idx_out) return PRUNER_EINVAL;
    if (!aligned(score, 4) || !aligned(idx_out, 4) || (val_out && !aligned(val_out, 4))) return PRUNER_EINVAL;
    const int32_t n_sg = ctx.n_sg, k = ctx.k;
    const SegT* d_segs = static_cast<const SegT*>(ctx.d_segs);
    const SegsInMemory in_memory{d_segs};
    InlineSegs inl;
    if (ctx.inline_ok) memcpy(&inl, ctx.inline_segs, sizeof inl);
    if (ctx.tiny) {
#define PRUNER_TINY(PER) \
    do { \
        if (ctx.inline_ok) hipLaunchKernelGGL((topk_tiny_kernel<PER, InlineSegs>), dim3(n_sg), dim3(kTinyThreads), 0, st, score, inl, k, idx_out, val_out); \
        else hipLaunchKernelGGL((topk_tiny_kernel<PER, SegsInMemory>), dim3(n_sg), dim3(kTinyThreads), 0, st, score, in_memory, k, idx_out, val_out); \
    } while (0)
        if (ctx.longest <= 2 * kTinyThreads) PRUNER_TINY(2);
        else if (ctx.longest <= 8 * kTinyThreads) PRUNER_TINY(8);
        else if (ctx.longest <= 16 * kTinyThreads) PRUNER_TINY(16);
        else PRUNER_TINY(kTinyPer);
#undef PRUNER_TINY
        PRUNER_LAUNCH_CHECK();
        return PRUNER_OK;
    }

    const int share = ctx.share;
    const bool sort = ctx.sort;
    const dim3 pickers((unsigned)((n_sg * share + kXcds - 1) / kXcds * kXcds));
#define PRUNER_PICK(LEVELS, TABLE, SEGS, GHIST, COPIES) \
    hipLaunchKernelGGL((sort ? pick_kernel<LEVELS, true, TABLE> : pick_kernel<LEVELS, false, TABLE>), pickers, dim3(kBigThreads), 0, st, score, SEGS, n_sg, (int)ctx.n, k, share, (Maxima{ctx.d_max16, ctx.d_max64, ctx.d_max256}), GHIST, COPIES, idx_out, val_out)
    if (ctx.levels || ctx.blocks_route) {
        if (!noted) {
            const int64_t most = (ctx.longest + kMaximaChunk - 1) / kMaximaChunk;
            const dim3 grid = most * n_sg <= ctx.blocks + kMaximaSpare ? dim3((unsigned)most, (unsigned)n_sg) : dim3((unsigned)ctx.blocks);
            if (ctx.inline_ok) hipLaunchKernelGGL(maxima_kernel<InlineSegs>, grid, dim3(256), 0, st, score, inl, n_sg, ctx.d_max16, ctx.d_max64, ctx.d_max256);
            else hipLaunchKernelGGL(maxima_kernel<SegsInMemory>, grid, dim3(256), 0, st, score, in_memory, n_sg, ctx.d_max16, ctx.d_max64, ctx.d_max256);
            PRUNER_LAUNCH_CHECK();
        }
        if (ctx.blocks_route) {
            static_assert(kBlocksSegments <= kInlineSegs, "the segment table travels with the launches");
            PartList* const parts = static_cast<PartList*>(ctx.d_parts);
            hipLaunchKernelGGL(block_lists_kernel<InlineSegs>, dim3((unsigned)(n_sg * kParts)), dim3(kBigThreads), 0, st, score, inl, (int)ctx.n, k, ctx.d_max256, parts);
            PRUNER_LAUNCH_CHECK();
            hipLaunchKernelGGL((sort ? pick_parts_kernel<true, InlineSegs> : pick_parts_kernel<false, InlineSegs>), pickers, dim3(kBigThreads), 0, st, score, inl, n_sg, k, share, parts, idx_out, val_out);
            PRUNER_LAUNCH_CHECK();
            return PRUNER_OK;
        }
        if (ctx.inline_ok) PRUNER_PICK(true, InlineSegs, inl, nullptr, 0);
        else PRUNER_PICK(true, SegsInMemory, in_memory, nullptr, 0);
        PRUNER_LAUNCH_CHECK();
        return PRUNER_OK;
    }
    if (ctx.pick && !ctx.digits) {
        if (ctx.inline_ok) PRUNER_PICK(false, InlineSegs, inl, nullptr, 0);
        else PRUNER_PICK(false, SegsInMemory, in_memory, nullptr, 0);
        PRUNER_LAUNCH_CHECK();
        return PRUNER_OK;
    }

    SelState* d_state = static_cast<SelState*>(ctx.d_state);
    Stage* d_stage = static_cast<Stage*>(ctx.d_stage);
    const int R = ctx.copies;
    const int64_t span = ctx.span;
    const size_t per_pass = (size_t)n_sg * kBins;
    uint32_t *hist0 = ctx.d_hist, *hist1 = ctx.d_hist + (size_t)R * per_pass, *hist2 = hist1 + per_pass;
    const dim3 chunks((unsigned)ctx.blocks);
    // (the draft kernel writes the block maxima when it counts the first digit)
    uint32_t* const block_max = ctx.d_max256;
    if (!noted) {
        hipLaunchKernelGGL(hist0_kernel, chunks, dim3(kBigThreads), 0, st, score, d_segs, n_sg, span, R, hist0, block_max);
        PRUNER_LAUNCH_CHECK();
    }
    if (ctx.pick) {
        if (ctx.longest > kCountMax) hipLaunchKernelGGL((sort ? pick_long_kernel<true> : pick_long_kernel<false>), pickers, dim3(kBigThreads), 0, st, score, d_segs, n_sg, (int)ctx.n, k, share, hist0, R, idx_out, val_out);
        else PRUNER_PICK(false, SegsInMemory, in_memory, hist0, R);
        PRUNER_LAUNCH_CHECK();
        return PRUNER_OK;
    }
#undef PRUNER_PICK
    if (ctx.lists) {
        hipLaunchKernelGGL(list_kernel, chunks, dim3(kBigThreads), 0, st, score, d_segs, n_sg, span, R, k, hist0, hist1, hist2, d_stage);
        PRUNER_LAUNCH_CHECK();
        hipLaunchKernelGGL((sort ? pick_lists_kernel<true> : pick_lists_kernel<false>), pickers, dim3(kBigThreads), 0, st, score, d_segs, n_sg, R, k, share, (int)span, hist0, hist1, hist2, d_stage,
                           ctx.blocks, idx_out, val_out);
        PRUNER_LAUNCH_CHECK();
        return PRUNER_OK;
    }
    if (block_max) hipLaunchKernelGGL(funnel_kernel<true>, chunks, dim3(kBigThreads), 0, st, score, d_segs, n_sg, span, R, k, hist0, hist1, d_state, d_stage, block_max);
    else hipLaunchKernelGGL(funnel_kernel<false>, chunks, dim3(kBigThreads), 0, st, score, d_segs, n_sg, span, R, k, hist0, hist1, d_state, d_stage, block_max);
    PRUNER_LAUNCH_CHECK();
    hipLaunchKernelGGL(refine_kernel, chunks, dim3(kBigThreads), 0, st, score, d_segs, n_sg, span, hist1, hist2, d_state, d_stage);
    PRUNER_LAUNCH_CHECK();
    hipLaunchKernelGGL(settle_kernel, chunks, dim3(kBigThreads), 0, st, score, d_segs, n_sg, span, k, hist2, d_state, d_stage);
    PRUNER_LAUNCH_CHECK();
    hipLaunchKernelGGL(gather_sort_kernel, dim3((unsigned)(n_sg * share)), dim3(kSmallThreads), 0, st, score, d_segs, n_sg, ctx.blocks, span,
                       d_state, d_stage, k, share, idx_out, val_out);
    PRUNER_LAUNCH_CHECK();
    return PRUNER_OK;
}

}  // namespace pruner

using namespace pruner;

extern "C" int pruner_topk(const float* score, const int64_t* seg_off, int32_t n_sg, int32_t k, int32_t* idx_out, float* val_out,
                           void* workspace, size_t workspace_bytes, void* stream)
{
    if (!score || !idx_out) return PRUNER_EINVAL;
    if (!aligned(score, 4) || !aligned(idx_out, 4) || (val_out && !aligned(val_out, 4))) return PRUNER_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    TopkCtx ctx;
    const int rc = topk_prepare(seg_off, n_sg, k, workspace, workspace_bytes, st, &ctx, nullptr, true, false);
    if (rc) return rc;
    return topk_finish(ctx, score, seg_off, idx_out, val_out, false, st);
}


// ---- selection without a workspace argument -------------------------------------------------------------------------
// The scratch of pruner_topk (segment table, selection state, digit histograms, staging slots) in a file-scope device
// array, for callers that cannot allocate.  One array per device, held until the process ends; every call on a device
// uses it, so calls that overlap on one device race.  Nothing in it has to survive between calls: the histograms are
// cleared by the call's first launch, every other part is written before it is read.
namespace {
constexpr size_t kStaticScratchBytes = (size_t)8 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
void* g_scratch_ptr[kMaxDevices];   // the array's device address on each device, looked up once
}  // namespace

extern "C" int pruner_topk_static(const float* score, const int64_t* seg_off, int32_t n_sg, int32_t k, int32_t* idx_out, float* val_out,
                                  void* stream)
{
    if (!score || !idx_out || !seg_off) return PRUNER_EINVAL;
    if (!aligned(score, 4) || !aligned(idx_out, 4) || (val_out && !aligned(val_out, 4))) return PRUNER_EINVAL;
    if (n_sg > PRUNER_STATIC_MAX_SEGMENTS) return PRUNER_EINVAL;
    static_assert(PRUNER_STATIC_MAX_SEGMENTS <= kFewSegs, "the segment table of a static call is built on the stack");
    int64_t longest = 0;
    const int bad = topk_check(seg_off, n_sg, k, &longest);
    if (bad) return bad;
    // the scratch a call of this size needs (it grows with the segment count, hardly with n)
    if (layout(seg_off[n_sg], n_sg, k, false).total > kStaticScratchBytes) return PRUNER_EWORKSPACE;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return PRUNER_EHIP;
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return PRUNER_EHIP;
        g_scratch_ptr[dev] = p;
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    TopkCtx ctx;
    const int rc = topk_prepare(seg_off, n_sg, k, g_scratch_ptr[dev], kStaticScratchBytes, st, &ctx, nullptr, false, false);
    if (rc) return rc;
    return topk_finish(ctx, score, seg_off, idx_out, val_out, false, st);
}
