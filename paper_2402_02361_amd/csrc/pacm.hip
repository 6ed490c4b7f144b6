// The whole Pattern-aware Transformer of the verify stage (Sec. 4.2): statement branch, self-attention over the
// temporal dataflow blocks, concatenation, linear head.  The paper's figure with the dimensions is lost; the model
// taken here (hidden 256, embedding 64, one attention head and layer with a residual connection, sum pooling, one
// hidden head layer):
//   statement s < n_stmt:  h1 = relu(W1 x_s + b1);  h2 = relu(W2 h1 + b2);          v_s = sum_s h2          (256)
//   block i < n_blk:       e_i = relu(We d_i + be);  q_i, k_i, v_i = Wq e_i, Wk e_i, Wv e_i
//                          a_ij = softmax_j(q_i . k_j / 8),  o_i = sum_j a_ij v_j
//                          z_i = e_i + Wo o_i;                                     v_d = sum_i z_i         (64)
//   head:                  g = relu(Wh [v_s ; v_d] + bh);  y = wo . g + bo
// Every operand of a matrix product is bfloat16 (inputs, e, q, k, v, o, h1, h2, the pooled vectors), accumulation is
// binary32, the softmax is binary32.
//
// Three launches:
//   pacm_stmt_kernel   the two statement layers on the matrix cores, tiles of 64 valid rows that hold whole candidates,
//                      the sum over a candidate's rows as one more matrix product; a wavefront owns 64 hidden units and
//                      keeps its W1/W2 slices in registers
//   pacm_flow_kernel   the dataflow branch, a wavefront per tile of 32 valid blocks that hold whole candidates, the chain
//                      from the features to the pooled vector in registers
//   pacm_head_kernel   the head's hidden layer on the matrix cores (64 candidates per tile) and its output dot product
// The pooled vectors travel through the workspace as the bfloat16 operands that the head's layer takes.
//
// Measured, before = eight padded slots per candidate in either branch and binary32 pooled vectors (statement counts 3..8,
// blocks 0..5): 131,072 candidates: statement kernel 345 -> 180 us, dataflow 170 -> 55, head 43 -> 28, the call 512-560 -> 246;
// 8,192 candidates: 29.8 -> 17.6, 23.7 -> 12.3, 10.7 -> 9.6, the call 60.4 -> 37.1.
#include "common.h"
#include "mfma_tile.h"

namespace pruner {
namespace {

using namespace tile;

constexpr int kF = PRUNER_FEAT_DIM;      // 164
constexpr int kS = PRUNER_MAX_STMT;      // 8
constexpr int kH = PRUNER_HIDDEN;        // 256
constexpr int kD = PRUNER_FLOW_DIM;      // 23
constexpr int kT = PRUNER_MAX_BLOCKS;    // 8
constexpr int kE = PRUNER_EMBED;         // 64
constexpr int kU = kH + kE;              // 320: the head's input
constexpr int kTM = 64;                  // rows per tile
constexpr int kK1 = 176;                 // 164 padded to a multiple of the MFMA depth 16
constexpr int kXs = kK1 + 8;             // LDS row strides in bfloat16 elements (rows stay 16-byte aligned)
constexpr int kHs = kH + 8;
constexpr int kUs = kU + 8;
constexpr int kThreads = 256;
constexpr int kF4 = kF / 4;              // float4 per feature row (41)
static_assert(kS == 8 && kT == 8 && kE == 64 && kTM == 64, "the lane arithmetic below assumes these");

__device__ __forceinline__ int clamp8(int v) { return v < 0 ? 0 : v > 8 ? 8 : v; }

// x = hi + mid + lo exactly, each a bfloat16 (3 x 8 significand bits; an infinity or a NaN is its own first piece)
struct Pieces {
    uint32_t hi, mid, lo;   // bit patterns
};
__device__ __forceinline__ Pieces split3(float x)
{
    const __bf16 hi = (__bf16)x;
    const float rest = x - (float)hi;
    const __bf16 mid = (__bf16)rest;
    const __bf16 lo = (__bf16)(rest - (float)mid);
    return Pieces{__builtin_bit_cast(uint16_t, hi), __builtin_bit_cast(uint16_t, mid), __builtin_bit_cast(uint16_t, lo)};
}

// Registers 8 q .. 8 q + 7 of a product as the operand of the next one: rounded to bfloat16 in pairs (with ReLU or without),
// or as three operands whose sum they are.
__device__ __forceinline__ bf16x8 relu_fragment(const floatx16& a, int q)
{
    const u32x4 f = {relu_bf16x2(a[8 * q], a[8 * q + 1]), relu_bf16x2(a[8 * q + 2], a[8 * q + 3]), relu_bf16x2(a[8 * q + 4], a[8 * q + 5]),
                     relu_bf16x2(a[8 * q + 6], a[8 * q + 7])};
    return __builtin_bit_cast(bf16x8, f);
}
__device__ __forceinline__ uint32_t bf16x2_of(float a, float b) { return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{a, b}), bf16x2)); }
__device__ __forceinline__ bf16x8 plain_fragment(const floatx16& a, int q)
{
    const u32x4 f = {bf16x2_of(a[8 * q], a[8 * q + 1]), bf16x2_of(a[8 * q + 2], a[8 * q + 3]), bf16x2_of(a[8 * q + 4], a[8 * q + 5]),
                     bf16x2_of(a[8 * q + 6], a[8 * q + 7])};
    return __builtin_bit_cast(bf16x8, f);
}
__device__ __forceinline__ void split_fragment(const floatx16& a, int q, bf16x8 (&piece)[3])
{
    u32x4 f[3];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        float x = a[8 * q + 2 * p], y = a[8 * q + 2 * p + 1];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            f[k][p] = bf16x2_of(x, y);
            x -= __uint_as_float(f[k][p] << 16);
            y -= __uint_as_float(f[k][p] & 0xFFFF0000u);
        }
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) piece[k] = __builtin_bit_cast(bf16x8, f[k]);
}
// What this wavefront's lanes wrote to LDS before is there for its other lanes after (LDS serves a wavefront in order; this
// keeps the compiler's order).
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// This wavefront's 64 rows of a [256][K] bfloat16 matrix as MFMA A operands: lane (l32, half) takes, per 32-row block
// and 16-deep step, the 16 bytes at row 64 wave + 32 nt + l32, depth 16 ks + 8 half.  FULL depth steps only.
template <int KS, int KFULL, typename V>
__device__ __forceinline__ void load_slices(bf16x8 (&wr)[2][KS], const uint16_t* __restrict__ W, int row_elems, int wave, int l32, int half)
{
    typedef V vec_t;
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
        const uint16_t* r = W + (size_t)(64 * wave + 32 * nt + l32) * row_elems + 8 * half;
#pragma unroll
        for (int ks = 0; ks < KFULL; ++ks) wr[nt][ks] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const vec_t*>(r + 16 * ks));
    }
}

// ---- pooling on the matrix cores -------------------------------------------------------------------------------------
// A layer computed with the rows as the A operand leaves a lane one output unit (l32) of 16 rows: register i is row
// 8 (i / 4) + 4 half + i % 4 of its 32-row block.  Rounded to bfloat16 in pairs, registers 8 q .. 8 q + 7 are, as they
// stand, one operand of a further MFMA whose depth is 16 of those rows; the other operand is the 0/1 matrix that says
// which candidate a row belongs to.  The product holds the sums over each candidate's rows, whatever their number, for
// 32 units x 32 candidates, a lane holding 16 units of ONE candidate.  Products with 1 are exact and the sums are binary32.

// A tile takes whole candidates; `rows` of lane (l32, half) is the set of rows of its l32-th candidate, one bit per row.
// Fragment q of the 0/1 matrix: rows 16 q + 8 (j / 4) + 4 half + j % 4 for j = 0..7.
__device__ __forceinline__ bf16x8 member_fragment(uint32_t rows32, int q, int half)
{
    const uint32_t n0 = rows32 >> (16 * q + 4 * half), n1 = rows32 >> (16 * q + 8 + 4 * half);
    auto two = [](uint32_t b) { return (uint32_t)__umul24((b & 1u) | ((b & 2u) << 15), 0x3F80u); };   // 1.0 where the bit is set
    const u32x4 f = {two(n0), two(n0 >> 2), two(n1), two(n1 >> 2)};
    return __builtin_bit_cast(bf16x8, f);
}
// the lowest n bits, n = 0..64
__device__ __forceinline__ uint64_t low_bits(uint32_t n) { return n >= 64 ? ~0ull : (1ull << n) - 1ull; }

// The lane's 16 units (block of 32, registers of one product) of its candidate, rounded, to the pooled vectors.
__device__ __forceinline__ void store_pooled(const floatx16& acc, int g, uint16_t* __restrict__ to)   // four units: 8 g + 4 half ..
{
    const f32x2 lo = {acc[4 * g + 0], acc[4 * g + 1]}, hi = {acc[4 * g + 2], acc[4 * g + 3]};
    u32x2 o;
    o[0] = __builtin_bit_cast(uint32_t, __builtin_convertvector(lo, bf16x2));
    o[1] = __builtin_bit_cast(uint32_t, __builtin_convertvector(hi, bf16x2));
    *reinterpret_cast<u32x2*>(to) = o;
}

// ---- statement branch ------------------------------------------------------------------------------------------------
// Bound: the matrix cores (and the chip's power) at scale, weights and first rows on their way for small sets.  Tiles of
// 64 valid rows: a tile takes as many whole candidates as fit (at most 32), so the rows beyond n_stmt cost nothing, and a
// candidate never straddles.  The candidates of a workgroup are groups of neighbours, interleaved over the workgroups as
// in verify_mlp.hip; so are the weights in registers, b1 in the depth padding and the two halves of a tile half a layer
// apart.

constexpr int kRowThreads = 8;                                   // threads that share a feature row: 128 contiguous bytes per request
constexpr int kXPass = kTM / (kThreads / kRowThreads);           // passes over the tile's rows (2)
constexpr int kXCols = (kF4 + kRowThreads - 1) / kRowThreads;    // float4 a thread fetches per row (6)
constexpr int kXLoads = kXPass * kXCols;                         // float4 a thread fetches per tile (12)
constexpr int kLocalCap = 2048;                                  // most candidates one workgroup takes in a launch
constexpr int kGroupMin = 8, kGroupMax = 64;                     // neighbouring candidates that go to one workgroup together

__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(1, 1)))
pacm_stmt_kernel(const float* __restrict__ feat, const int32_t* __restrict__ n_stmt, int32_t n_d, int group_log, const uint16_t* __restrict__ W1,
                 const float* __restrict__ b1, const uint16_t* __restrict__ W2, const float* __restrict__ b2, uint16_t* __restrict__ v_s)
{
    __shared__ __attribute__((aligned(16))) __bf16 arena[kTM * kXs + kTM * kHs];
    __shared__ uint16_t before[kLocalCap + 64 + 2];   // valid rows of this workgroup's candidates 0..l-1 (at most 8 x kLocalCap)
    __shared__ int32_t row_src[kTM];                  // what the rows of one tile are: candidate * 8 + statement, or -1
    __shared__ uint32_t scan_tot[4];
    __shared__ uint32_t tainted[kLocalCap / 32];      // tiles to do again, by their first candidate
    __bf16* X = arena;                   // feature tile, bfloat16 [kTM][kXs]
    __bf16* H1 = arena + kTM * kXs;      // first hidden layer of the tile [kTM][kHs]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int half = lane >> 5, l32 = lane & 31;

    // this workgroup's candidates: groups b, b + G, ... of 2^group_log neighbours
    const int n_groups = (n_d + (1 << group_log) - 1) >> group_log, my_first = (int)blockIdx.x, group_stride = (int)gridDim.x;
    const int my_groups = my_first < n_groups ? (n_groups - my_first + group_stride - 1) / group_stride : 0;
    const bool owns_last = my_groups > 0 && my_first + (my_groups - 1) * group_stride == n_groups - 1;
    const int n_local = (my_groups << group_log) - (owns_last ? (n_groups << group_log) - n_d : 0);
    auto global_of = [&](int l) -> int { return ((((l >> group_log) * group_stride + my_first)) << group_log) + (l & ((1 << group_log) - 1)); };

    // weights: W1's rows end at depth 164; the last step holds its last four entries and b1 as three bfloat16 pieces
    // (b = hi + mid + lo exactly), which meet the 1, 1, 1 that the feature tile holds at depths 164..166
    static_assert(kK1 / 16 == kF / 16 + 1 && kF % 16 == 4, "W1's last depth step holds four entries");
    bf16x8 w1r[2][kK1 / 16], w2r[2][kH / 16];
    typedef u32x4 u32x4_a8 __attribute__((aligned(8)));   // W1's rows are 328 bytes
    load_slices<kK1 / 16, kF / 16, u32x4_a8>(w1r, W1, kF, wave, l32, half);
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
        const int n = 64 * wave + 32 * nt + l32;
        const u32x2 tail = *reinterpret_cast<const u32x2*>(W1 + (size_t)n * kF + 16 * (kF / 16));
        u32x4 last = {0u, 0u, 0u, 0u};
        const Pieces b = split3(b1[n]);
        last[0] = half == 0 ? tail[0] : 0u;
        last[1] = half == 0 ? tail[1] : 0u;
        last[2] = half == 0 ? (b.hi | (b.mid << 16)) : 0u;
        last[3] = half == 0 ? b.lo : 0u;
        w1r[nt][kF / 16] = __builtin_bit_cast(bf16x8, last);
    }
    const float b2_mine[2] = {b2[64 * wave + l32], b2[64 * wave + 32 + l32]};

    {   // row numbering: exclusive scan of the statement counts, a run of `per` candidates per thread
        for (int l = threadIdx.x; l < n_local; l += kThreads) before[l] = (uint16_t)clamp8(n_stmt[global_of(l)]);
        __syncthreads();
        const int per = ((n_local + kThreads - 1) / kThreads) | 1;
        const int c_lo = (int)threadIdx.x * per < n_local ? (int)threadIdx.x * per : n_local;
        const int c_hi = c_lo + per < n_local ? c_lo + per : n_local;
        uint32_t mine = 0;
        for (int c = c_lo; c < c_hi; ++c) mine += before[c];
        const uint32_t incl = wave_inclusive_sum(mine);
        if (lane == 63) scan_tot[wave] = incl;
        __syncthreads();
        uint32_t run = incl - mine, total = 0;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            run += w < wave ? scan_tot[w] : 0u;
            total += scan_tot[w];
        }
        for (int c = c_lo; c < c_hi; ++c) {
            const uint32_t v = before[c];
            before[c] = (uint16_t)run;
            run += v;
        }
        for (int i = threadIdx.x; i < 64 + 2; i += kThreads) before[n_local + i] = (uint16_t)total;
        __syncthreads();
    }

    // A tile, as every wavefront sees it: candidates start .. start + count - 1 of this workgroup; lane (l32, half) holds
    // the first and last + 1 row and the place of the l32-th of them (-1 past the last).
    struct Tile {
        int start, count;
        uint32_t first, end;
        int cand;
    };
    int stop = n_local, most = 32;   // tiles end before candidate `stop` and take at most `most` candidates
    auto tile_at = [&](int start) {
        Tile t;
        t.start = start;
        const int i = start + l32 < n_local ? start + l32 : n_local;
        const uint32_t b0 = before[i], b1v = before[i + 1];
        const uint32_t base = (uint32_t)__builtin_amdgcn_readfirstlane((int)b0);
        t.first = b0 - base;
        t.end = b1v - base;
        const bool in = start + l32 < stop && l32 < most && t.end <= (uint32_t)kTM;
        t.count = (int)__popcll(__ballot(in) & 0xFFFFFFFFull);   // (the counts grow, so the candidates that fit are the first ones)
        t.cand = in ? global_of(start + l32) : -1;
        t.first = in ? t.first : 0u;
        t.end = in ? t.end : 0u;
        return t;
    };
    auto rows_of = [&](const Tile& t) { return low_bits(t.end) & ~low_bits(t.first); };
    auto write_rows = [&](const Tile& t) {   // by one wavefront
        const int used = t.count > 0 ? __builtin_amdgcn_readlane((int)t.end, t.count - 1) : 0;
        if (lane >= used) row_src[lane] = -1;
        if (half == 0) {
#pragma unroll
            for (int st = 0; st < kS; ++st)
                if (t.first + (uint32_t)st < t.end) row_src[t.first + (uint32_t)st] = t.cand * kS + st;
        }
    };

    // features: as in verify_mlp.hip, twelve pieces per thread, requested two stages before they are parked; rows past the
    // tile's last become zero rows
    f32x4 xr[kXLoads];
    int fetch_src[kXPass];
    const int f_sub = threadIdx.x & (kRowThreads - 1), f_row = threadIdx.x / kRowThreads;
    auto fetch_read = [&]() {
#pragma unroll
        for (int ps = 0; ps < kXPass; ++ps) fetch_src[ps] = row_src[f_row + ps * (kThreads / kRowThreads)];
    };
    auto fetch_issue = [&](int i) {
        const int ps = i / kXCols, col = f_sub + kRowThreads * (i % kXCols);
        const int sr = fetch_src[ps];
        xr[i] = *reinterpret_cast<const f32x4*>(feat + (size_t)(sr < 0 ? 0 : sr) * kF + 4 * (col < kF4 ? col : kF4 - 1));
    };
    auto park_piece = [&](int i) {
        const int ps = i / kXCols, col = f_sub + kRowThreads * (i % kXCols);
        const f32x2 lo = {xr[i][0], xr[i][1]}, hi = {xr[i][2], xr[i][3]};
        const uint32_t there = fetch_src[ps] < 0 ? 0u : ~0u;
        u32x2 o;
        o[0] = __builtin_bit_cast(uint32_t, __builtin_convertvector(lo, bf16x2)) & there;
        o[1] = __builtin_bit_cast(uint32_t, __builtin_convertvector(hi, bf16x2)) & there;
        *reinterpret_cast<u32x2*>(&X[(f_row + ps * (kThreads / kRowThreads)) * kXs + (col < kF4 ? 4 * col : kK1)]) = o;   // depth 176..179 is never read
    };

    // the second layer's matrix: not needed before the first tile's second layer
    load_slices<kH / 16, kH / 16, u32x4>(w2r, W2, kH, wave, l32, half);
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)   // weights in the accumulation registers (see verify_mlp.hip)
#pragma unroll
        for (int ks = 0; ks < kK1 / 16; ++ks) asm volatile("" : "+a"(w1r[nt][ks]));
    // the padding of the feature tile (depth 164..183) is written once: 1, 1, 1 (times the three pieces of b1), then zeros
    for (int q = threadIdx.x; q < kTM * ((kXs - kF) / 4); q += kThreads) {
        const int r = q / ((kXs - kF) / 4), j = q % ((kXs - kF) / 4);
        *reinterpret_cast<uint2*>(&X[r * kXs + kF + 4 * j]) = j == 0 ? make_uint2(0x3F803F80u, 0x00003F80u) : make_uint2(0, 0);
    }
    for (int i = threadIdx.x; i < kLocalCap / 32; i += kThreads) tainted[i] = 0u;
    floatx16 b2r[2];
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
        for (int i = 0; i < 16; ++i) b2r[nt][i] = b2_mine[nt];

    floatx16 acc0[2], acc1[2];   // rows 0..31 and 32..63
    floatx16 pooled[2];          // sums of the tile in the making: units 64 wave + 32 nt + .. of the lane's candidate
    uint32_t pk[16];             // a half's second hidden layer, pairs of neighbouring rows
    bf16x8 member[4];            // the 0/1 matrix of the tile being pooled: 16 rows each
    uint32_t top;                // the largest of a half's activations (a lane's pairs), as 16-bit integers
    bool special;                // the tile being pooled holds an infinity or a NaN
    int pool_start, pool_count;
    uint32_t pool_to;            // where the lane's candidate goes (bytes from v_s), or past the end of the buffer: no store
    constexpr uint32_t kNowhere = 0xFFFF0000u;
    const auto out = __builtin_amdgcn_make_buffer_rsrc(v_s, 0, n_d * kH * 2, 0x00027000);

    auto pack_pair = [&](const floatx16(&acc)[2], int pair) {
        const int nt = pair >> 3, j = pair & 7;
        pk[pair] = relu_bf16x2(acc[nt][2 * j], acc[nt][2 * j + 1]);
        // (not negative, so the order of the bit patterns is the order of the values, infinity and NaN last)
        top = pair == 0 ? pk[0] : __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(i16x2, top), __builtin_bit_cast(i16x2, pk[pair])));
    };
    auto is_special = [&]() { return __ballot((top & 0xFFFFu) >= 0x7F80u || (top >> 16) >= 0x7F80u) != 0ull; };
    auto pool_mfma = [&](int hh, int q) {   // q = 2 nt + hq
        const u32x4 h = {pk[4 * q], pk[4 * q + 1], pk[4 * q + 2], pk[4 * q + 3]};
        if (hh == 0 && (q & 1) == 0) {
            floatx16 zero;
#pragma unroll
            for (int i = 0; i < 16; ++i) zero[i] = 0.f;
            pooled[q >> 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, h), member[2 * hh + (q & 1)], zero, 0, 0, 0);
        } else {
            pooled[q >> 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, h), member[2 * hh + (q & 1)], pooled[q >> 1], 0, 0, 0);
        }
    };
    auto pool_store = [&](int piece) {   // four units of the lane's candidate
        const int nt = piece >> 2, g = piece & 3;
        const u32x2 o = {bf16x2_of(pooled[nt][4 * g + 0], pooled[nt][4 * g + 1]), bf16x2_of(pooled[nt][4 * g + 2], pooled[nt][4 * g + 3])};
        __builtin_amdgcn_raw_buffer_store_b64(o, out, (int)(pool_to + 2u * (uint32_t)(32 * nt + 8 * g)), 0, 0);
    };
    // 0 times an infinity or a NaN of one candidate would reach the others of its tile: such a tile is noted and done again
    // when the others are through, one candidate at a time.
    auto note_special = [&]() {
        if (special && pool_count > 1 && lane == 0) atomicOr(&tainted[pool_start >> 5], 1u << (pool_start & 31));
    };

    int begin = 0, again = 0;   // candidates from `again` on may belong to noted tiles (second and later rounds)
    for (;;) {
        special = false;
        pool_start = pool_count = 0;
        pool_to = kNowhere;
        top = 0u;
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc0[nt][i] = acc1[nt][i] = pooled[nt][i] = 0.f;
#pragma unroll
        for (int q = 0; q < 4; ++q) member[q] = __builtin_bit_cast(bf16x8, u32x4{0u, 0u, 0u, 0u});
        Tile cur = tile_at(begin);
        if (wave == 0) write_rows(cur);
        __syncthreads();
        fetch_read();
#pragma unroll
        for (int i = 0; i < kXLoads; ++i) fetch_issue(i);
        Tile nxt = tile_at(cur.start + cur.count);
        __syncthreads();   // everyone has read the first tile's rows
        if (wave == 0) write_rows(nxt);
#pragma unroll
        for (int i = 0; i < kXLoads; ++i) park_piece(i);
        __syncthreads();
        fetch_read();
#pragma unroll
        for (int i = 0; i < kXLoads; ++i) fetch_issue(i);

        // A tile in four stages, each a layer of one half of the rows with other work between its MFMAs.  At the loop's head
        // X holds this tile's rows and the next tile's are on their way to registers.
        while (cur.count > 0) {
            // layer 1, rows 0..31.  Meanwhile: the sums of the previous tile's rows 32..63.
            layer_from<kK1 / 16>(acc0, nullptr, w1r, X, kXs, l32, half, [&](int i) {
                if (i < 8) {
                    pack_pair(acc1, 2 * i);
                    pack_pair(acc1, 2 * i + 1);
                    if (i & 1) pool_mfma(1, i >> 1);
                }
                if (i == 8) special = special || is_special();
            });
            // layer 1, rows 32..63.  Meanwhile: hidden layer 1 of rows 0..31 to LDS, the previous tile's sums to memory.
            layer_from<kK1 / 16>(acc1, nullptr, w1r, X + 32 * kXs, kXs, l32, half, [&](int i) {
                if (i >= 4 && i < 20 && !(i & 1)) park_hidden(acc0, (i - 4) >> 1, H1, kHs, wave, l32, half);
                if (i >= 1 && i < 17 && (i & 1)) pool_store(i >> 1);
                if (i == 17) note_special();
                if (i == 18) {
                    pool_start = cur.start;
                    pool_count = cur.count;
                    pool_to = cur.cand >= 0 ? 2u * ((uint32_t)cur.cand * kH + 64 * wave + 4 * half) : kNowhere;
                }
                if (i >= 18) member[i - 18] = member_fragment((uint32_t)(rows_of(cur) >> (i >= 20 ? 32 : 0)), (i - 18) & 1, half);
            });
            __syncthreads();   // rows 0..31 of H1 complete; X no longer read
            // layer 2, rows 0..31.  Meanwhile: hidden layer 1 of rows 32..63 and the next tile's features to LDS, and what
            // the rows of the tile after next are.
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)   // (no instruction: the register class, and in the first tile the wait for the matrix)
                asm volatile("" : "+a"(w2r[nt][0]), "+a"(w2r[nt][1]), "+a"(w2r[nt][2]), "+a"(w2r[nt][3]), "+a"(w2r[nt][4]), "+a"(w2r[nt][5]),
                                  "+a"(w2r[nt][6]), "+a"(w2r[nt][7]), "+a"(w2r[nt][8]), "+a"(w2r[nt][9]), "+a"(w2r[nt][10]), "+a"(w2r[nt][11]),
                                  "+a"(w2r[nt][12]), "+a"(w2r[nt][13]), "+a"(w2r[nt][14]), "+a"(w2r[nt][15]));
            static_assert(kH / 16 == 16, "the second layer's sixteen depth steps are listed above");
            Tile after = nxt;
            layer_rows<kH / 16>(acc0, b2r, w2r, H1, kHs, l32, half, [&](int i) {
                if (i & 1) {
                    if (i >= 2 * (kH / 16 - kXLoads)) park_piece((i - 2 * (kH / 16 - kXLoads)) >> 1);   // as late as the layer allows
                    return;
                }
                if (i < 16) park_hidden(acc1, i >> 1, H1 + 32 * kHs, kHs, wave, l32, half);
                if (i == 18) after = tile_at(nxt.start + nxt.count);
                if (i == 26 && wave == 0) write_rows(after);
            });
            __syncthreads();   // rows 32..63 of H1, X (the next tile's rows) and the rows' table complete
            // layer 2, rows 32..63.  Meanwhile: the sums of rows 0..31, and the requests for the rows of the tile after next.
            layer_rows<kH / 16>(acc1, b2r, w2r, H1 + 32 * kHs, kHs, l32, half, [&](int i) {
                if (!(i & 1) && i < 16) {
                    pack_pair(acc0, i);
                    pack_pair(acc0, i + 1);
                }
                if ((i & 3) == 3 && i < 16) pool_mfma(0, i >> 2);
                if (i == 0) fetch_read();
                if ((i & 1) && i < 2 * kXLoads) fetch_issue(i >> 1);
                if (i == 18) special = is_special();
            });
            cur = nxt;
            nxt = after;
        }
        // the last tile's second half
#pragma unroll
        for (int pair = 0; pair < 16; ++pair) pack_pair(acc1, pair);
#pragma unroll
        for (int q = 0; q < 4; ++q) pool_mfma(1, q);
        special = special || is_special();
#pragma unroll
        for (int piece = 0; piece < 8; ++piece) pool_store(piece);
        note_special();
        // the next noted tile, if there is one
        __syncthreads();
        int found = -1;
        for (int w = again >> 5; w < (n_local + 31) / 32 && found < 0; ++w) {
            const uint32_t bits = tainted[w] & (w == again >> 5 ? ~0u << (again & 31) : ~0u);
            if (bits) found = 32 * w + __builtin_ctz(bits);
        }
        if (found < 0) break;
        begin = again = found;
        stop = n_local;
        most = 32;
        const Tile t = tile_at(found);   // (the tile as it was: its first candidate names it)
        stop = found + t.count;
        most = 1;
        again = stop;
    }
}

// ---- dataflow branch -------------------------------------------------------------------------------------------------
// A wavefront works on tiles of 32 block slots: as many whole candidates as fit, so slots beyond n_blk cost nothing.  The
// whole chain stays in registers.  A layer computed transposed (weights as the A operand) leaves a lane 16 units of its
// row, computed straight (rows as the A operand) 16 rows of its unit; rounded in pairs, either is the operand of the next
// product as it stands, as long as the other operand numbers the depth the same way (the weight matrices are read in that
// order once).  So:
//   E (both ways) from the features; Q, K (units per lane) and V (rows per lane) from E; the scores with a query per lane and
//   its 32 keys over two lanes: keys of other candidates are masked, the softmax is lane-local but for one exchange; the
//   binary32 attention weights go to the matrix cores as three bfloat16 pieces (p = hi + mid + lo exactly, products exact,
//   binary32 sums); O rounded is the operand of Wo; Z = Wo O, in three pieces again, and E are summed over each candidate's
//   rows by the 0/1 matrix of the statement branch.
// 0 times an infinity or a NaN of one candidate would reach the others of its tile: a tile whose sums hold a NaN is done
// again candidate by candidate.
// Bound: vector instructions (the softmax, the pieces).  Eight slots per candidate, softmax and products with the weights on
// the vector ALU and every stage through LDS took 170 us where this takes 55 (131,072 candidates, 2.8 blocks on average).

constexpr int kFlowWaves = 4;                 // wavefronts per workgroup, each with tiles of its own
constexpr int kFlowThreads = 64 * kFlowWaves;
constexpr int kFlowGroup = 8;                 // neighbouring candidates that go to one wavefront together
constexpr int kFlowRows = 32;
constexpr int kFlowBlocksPerCu = 2;
constexpr int kDk = 32;                       // 23 padded to the MFMA depth: 1, 1, 1 meet the three pieces of the bias
constexpr int kFlowLocalCap = 1024;           // most candidates of one wavefront in a launch

__global__ void __launch_bounds__(kFlowThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
pacm_flow_kernel(const float* __restrict__ flow, const int32_t* __restrict__ n_blk, int32_t n_d, const uint16_t* __restrict__ We,
                 const float* __restrict__ be, const uint16_t* __restrict__ Wq, const uint16_t* __restrict__ Wk,
                 const uint16_t* __restrict__ Wv, const uint16_t* __restrict__ Wo, uint16_t* __restrict__ v_d)
{
    __shared__ uint8_t counts[kFlowWaves][kFlowLocalCap];       // blocks of the wavefront's candidates
    __shared__ uint32_t row_tab[kFlowWaves][2][kFlowRows];      // what the rows of a tile are (two tiles are in the making)
    __shared__ __attribute__((aligned(16))) u32x4 wv_lds[2][kE / 16][64], wo_lds[2][kE / 16][64];   // Wv's and Wo's fragments (registers hold the others)
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int half = lane >> 5, l32 = lane & 31;

    // this wavefront's candidates: groups W, W + NW, ... of kFlowGroup neighbours
    const int n_groups = (n_d + kFlowGroup - 1) / kFlowGroup, my_first = (int)blockIdx.x * kFlowWaves + wave, group_stride = (int)gridDim.x * kFlowWaves;
    const int my_groups = my_first < n_groups ? (n_groups - my_first + group_stride - 1) / group_stride : 0;
    const bool owns_last = my_groups > 0 && my_first + (my_groups - 1) * group_stride == n_groups - 1;
    const int n_local = my_groups * kFlowGroup - (owns_last ? n_groups * kFlowGroup - n_d : 0);
    auto global_of = [&](int l) -> int { return kFlowGroup * ((l / kFlowGroup) * group_stride + my_first) + l % kFlowGroup; };
    for (int l = lane; l < n_local; l += 64) counts[wave][l] = (uint8_t)clamp8(n_blk[global_of(l)]);

    // Weights, lane (l32, half): row 32 nt + l32 of the matrix.  We: eight depths 16 ks + 8 half + j (the features' order).
    // The others: the order in which a lane holds the units of a product, 16 ks + 8 (j / 4) + 4 half + j % 4.
    bf16x8 wer[2][kDk / 16], wqr[2][kE / 16], wkr[2][kE / 16];
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
        const int n = 32 * nt + l32;
        const Pieces b = split3(be[n]);
#pragma unroll
        for (int ks = 0; ks < kDk / 16; ++ks) {
            uint32_t pk[4];
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                uint32_t two[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const int k0 = 16 * ks + 8 * half + 2 * p + e;
                    two[e] = k0 < kD ? (uint32_t)We[n * kD + (k0 < kD ? k0 : 0)] : k0 == kD ? b.hi : k0 == kD + 1 ? b.mid : k0 == kD + 2 ? b.lo : 0u;
                }
                pk[p] = two[0] | (two[1] << 16);
            }
            wer[nt][ks] = __builtin_bit_cast(bf16x8, u32x4{pk[0], pk[1], pk[2], pk[3]});
        }
        auto fragment = [&](const uint16_t* W, int ks) {
            const uint16_t* r = W + (size_t)n * kE + 16 * ks + 4 * half;
            typedef u32x2 u32x2_a2 __attribute__((aligned(2)));
            const u32x2 lo = *reinterpret_cast<const u32x2_a2*>(r), hi = *reinterpret_cast<const u32x2_a2*>(r + 8);
            return u32x4{lo[0], lo[1], hi[0], hi[1]};
        };
#pragma unroll
        for (int ks = 0; ks < kE / 16; ++ks) {
            wqr[nt][ks] = __builtin_bit_cast(bf16x8, fragment(Wq, ks));
            wkr[nt][ks] = __builtin_bit_cast(bf16x8, fragment(Wk, ks));
            if (wave == 0) wo_lds[nt][ks][lane] = fragment(Wo, ks);
            if (wave == 1) wv_lds[nt][ks][lane] = fragment(Wv, ks);
        }
    }
    __syncthreads();   // (the only one: from here on every wavefront goes its own way)

    struct Tile {
        int start, count;
        uint32_t first, end;   // rows of the lane's (l32-th) candidate
        int cand;              // its place, -1 past the last
        uint32_t row;          // of the lane's (l32-th) row: first and end row of its candidate (8 bits each)
        f32x4 x[4];            // the lane's eight plus eight (half 1: eight) features of that row
    };
    auto zero16 = []() {
        floatx16 z;
#pragma unroll
        for (int i = 0; i < 16; ++i) z[i] = 0.f;
        return z;
    };
    // The tile from local candidate `start` on, at most `most` candidates; its features are requested.
    auto tile_at = [&](int start, int most, int buffer) {
        Tile t;
        t.start = start;
        const bool there = l32 < most && start + l32 < n_local;
        const uint32_t n = there && half == 0 ? counts[wave][start + l32] : 0u;
        const uint32_t upto = wave_inclusive_sum(n);   // (lanes 32..63 add nothing)
        const uint32_t n_all = (uint32_t)__shfl((int)n, l32, 64), upto_all = (uint32_t)__shfl((int)upto, l32, 64);
        const bool in = there && upto_all <= (uint32_t)kFlowRows;
        t.count = (int)__popcll(__ballot(in) & 0xFFFFFFFFull);
        t.cand = in ? global_of(start + l32) : -1;
        t.end = in ? upto_all : 0u;
        t.first = in ? upto_all - n_all : 0u;
        uint32_t* tab = row_tab[wave][buffer];
        if (half == 0) tab[l32] = 0u;
        wave_lds_fence();
        if (half == 0) {
#pragma unroll
            for (int b = 0; b < kT; ++b)   // (candidate of the tile, slot), first and end row; an empty row has first = end = 0
                if (t.first + (uint32_t)b < t.end) tab[t.first + (uint32_t)b] = t.first | (t.end << 8) | ((uint32_t)(l32 * kT + b) << 16);
        }
        wave_lds_fence();
        t.row = tab[l32];
        const int at = (int)(t.row >> 16);
        const int64_t src = (t.row & 0xFFFFu) == 0u ? 0 : (int64_t)global_of(start + at / kT) * kT + at % kT;
        typedef f32x4 f32x4_a4 __attribute__((aligned(4)));
        const float* r = flow + src * kD;
        t.x[0] = *reinterpret_cast<const f32x4_a4*>(r + 8 * half);
        t.x[1] = *reinterpret_cast<const f32x4_a4*>(r + 8 * half + 4);
        t.x[2] = *reinterpret_cast<const f32x4_a4*>(r + (half ? 8 : 16));
        t.x[3] = *reinterpret_cast<const f32x4_a4*>(r + (half ? 8 : 19));   // depths 20, 21, 22 are its last three
        return t;
    };

    int alone_until = 0;   // candidates before this one are done one by one
    Tile cur = tile_at(0, kFlowRows, 0);
    int buffer = 1;
    while (cur.count > 0) {
        const int next = cur.start + cur.count;
        const Tile nxt = tile_at(next, next < alone_until ? 1 : kFlowRows, buffer);
        buffer ^= 1;
        const uint32_t row_first = cur.row & 0xFFu, row_end = (cur.row >> 8) & 0xFFu;
        const bool row_there = row_end != 0u;
        // features, bfloat16, with 1, 1, 1 at depths 23..25
        bf16x8 d[2];
        {
            const uint32_t there = row_there ? ~0u : 0u;
            auto two = [](float a, float b) { return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{a, b}), bf16x2)); };
            const u32x4 d0 = {two(cur.x[0][0], cur.x[0][1]) & there, two(cur.x[0][2], cur.x[0][3]) & there, two(cur.x[1][0], cur.x[1][1]) & there,
                              two(cur.x[1][2], cur.x[1][3]) & there};
            u32x4 d1 = {two(cur.x[2][0], cur.x[2][1]) & there, two(cur.x[2][2], cur.x[2][3]) & there, two(cur.x[3][1], cur.x[3][2]) & there,
                        (two(cur.x[3][3], 0.f) & there) | 0x3F800000u};
            d1[0] = half ? 0x3F803F80u : d1[0];
            d1[1] = half ? 0u : d1[1];
            d1[2] = half ? 0u : d1[2];
            d1[3] = half ? 0u : d1[3];
            d[0] = __builtin_bit_cast(bf16x8, d0);
            d[1] = __builtin_bit_cast(bf16x8, d1);
        }
        const uint32_t my_rows = (uint32_t)(low_bits(cur.end) & ~low_bits(cur.first));
        bf16x8 member[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) member[q] = member_fragment(my_rows, q, half);

        floatx16 sum[2];   // v_d of the lane's candidate
        bf16x8 e[kE / 16];   // E, units per lane: operand ks = 2 nt + hq
        {
            floatx16 acc[2];
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) {   // rows per lane, summed right away
                acc[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(d[0], wer[nt][0], zero16(), 0, 0, 0);
                acc[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(d[1], wer[nt][1], acc[nt], 0, 0, 0);
            }
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
#pragma unroll
                for (int hq = 0; hq < 2; ++hq) {
                    const bf16x8 f = relu_fragment(acc[nt], hq);
                    sum[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, member[hq], hq == 0 ? zero16() : sum[nt], 0, 0, 0);
                }
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) {   // units per lane
                acc[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wer[nt][0], d[0], zero16(), 0, 0, 0);
                acc[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wer[nt][1], d[1], acc[nt], 0, 0, 0);
            }
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
#pragma unroll
                for (int hq = 0; hq < 2; ++hq) e[2 * nt + hq] = relu_fragment(acc[nt], hq);
        }
        floatx16 sc;
        {
            bf16x8 q[kE / 16], k[kE / 16];
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) {
                floatx16 aq = zero16(), ak = zero16();
#pragma unroll
                for (int ks = 0; ks < kE / 16; ++ks) {
                    aq = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wqr[nt][ks], e[ks], aq, 0, 0, 0);
                    ak = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wkr[nt][ks], e[ks], ak, 0, 0, 0);
                }
#pragma unroll
                for (int hq = 0; hq < 2; ++hq) {
                    q[2 * nt + hq] = plain_fragment(aq, hq);
                    k[2 * nt + hq] = plain_fragment(ak, hq);
                }
            }
            sc = zero16();
#pragma unroll
            for (int ks = 0; ks < kE / 16; ++ks) sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k[ks], q[ks], sc, 0, 0, 0);   // lane: query l32, keys 8 (i / 4) + 4 half + i % 4
        }
        bf16x8 v[2][2];   // V, rows per lane: [nt][hq]
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            floatx16 av = zero16();
#pragma unroll
            for (int ks = 0; ks < kE / 16; ++ks) av = __builtin_amdgcn_mfma_f32_32x32x16_bf16(e[ks], __builtin_bit_cast(bf16x8, wv_lds[nt][ks][lane]), av, 0, 0, 0);
#pragma unroll
            for (int hq = 0; hq < 2; ++hq) v[nt][hq] = plain_fragment(av, hq);
        }
        // softmax over the query's own keys
        float scale;
        {
            const uint32_t own = (uint32_t)(low_bits(row_end) & ~low_bits(row_first)) >> (4 * half);   // bit 8 (i / 4) + i % 4: register i's key is one
            float mx = -__builtin_inff();
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                sc[i] = (own >> (8 * (i / 4) + i % 4)) & 1u ? sc[i] * 0.125f : -__builtin_inff();
                mx = fmaxf(mx, sc[i]);
            }
            mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
            mx = row_there ? mx : 0.f;
            float den = 0.f;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                sc[i] = (own >> (8 * (i / 4) + i % 4)) & 1u ? expf(sc[i] - mx) : 0.f;
                den += sc[i];
            }
            den += __shfl_xor(den, 32, 64);
            scale = row_there ? 1.0f / den : 0.f;
        }
        // O^T[unit][query] = (sum over keys of V p) / den, the weights in three bfloat16 pieces
        bf16x8 o[kE / 16];
        {
            floatx16 acc[2];
#pragma unroll
            for (int hq = 0; hq < 2; ++hq) {
                bf16x8 piece[3];
                split_fragment(sc, hq, piece);
#pragma unroll
                for (int nt = 0; nt < 2; ++nt)
#pragma unroll
                    for (int p = 0; p < 3; ++p)
                        acc[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v[nt][hq], piece[2 - p], hq == 0 && p == 0 ? zero16() : acc[nt], 0, 0, 0);
            }
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) {
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[nt][i] *= scale;
#pragma unroll
                for (int hq = 0; hq < 2; ++hq) o[2 * nt + hq] = plain_fragment(acc[nt], hq);
            }
        }
        // Z = O Wo^T, rows per lane, in three pieces into the sums
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            floatx16 z = zero16();
#pragma unroll
            for (int ks = 0; ks < kE / 16; ++ks) z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(o[ks], __builtin_bit_cast(bf16x8, wo_lds[nt][ks][lane]), z, 0, 0, 0);
#pragma unroll
            for (int hq = 0; hq < 2; ++hq) {
                bf16x8 piece[3];
                split_fragment(z, hq, piece);
#pragma unroll
                for (int p = 0; p < 3; ++p) sum[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(piece[2 - p], member[hq], sum[nt], 0, 0, 0);
            }
        }
        float any = 0.f;   // NaN if one of the sums is (opposite infinities add up to one too: such a tile is merely done twice)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
            for (int i = 0; i < 16; ++i) any += sum[nt][i];
        if (cur.count > 1 && __ballot(any != any) != 0ull) {
            alone_until = next;
            cur = tile_at(cur.start, 1, buffer);
            buffer ^= 1;
            continue;
        }
        if (cur.cand >= 0) {
            uint16_t* to = v_d + (size_t)cur.cand * kE + 4 * half;
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
#pragma unroll
                for (int g = 0; g < 4; ++g) store_pooled(sum[nt], g, to + 32 * nt + 8 * g);
        }
        cur = nxt;
    }
}

// ---- head ------------------------------------------------------------------------------------------------------------
// The two 32-row halves of a tile run one after the other on the matrix cores; rounding, the output dot product (matrix cores
// as well, see last_layer_mfma) and the stores of one half, and the next tile's way into LDS, are issued between the MFMAs
// of the other.  Two tiles' operands in LDS: one barrier per tile.  Bound: memory at scale (640 bytes per candidate), weights
// and launch for small sets.

__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(1, 1)))
pacm_head_kernel(const uint16_t* __restrict__ v_s, const uint16_t* __restrict__ v_d, int32_t n_d, const uint16_t* __restrict__ Wh,
                 const float* __restrict__ bh, const uint16_t* __restrict__ wo, float bo, float* __restrict__ y)
{
    __shared__ __attribute__((aligned(16))) __bf16 U[2][kTM * kUs];   // a tile's concatenated pooled vectors
    __shared__ __attribute__((aligned(16))) float cst[kH];
    __shared__ __attribute__((aligned(16))) uint16_t wo_lds[kH];
    __shared__ float red[2][4][kTM];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int half = lane >> 5, l32 = lane & 31;
    const int n_tiles = (n_d + kTM - 1) / kTM;

    constexpr int kU8 = kU / 8;   // 16-byte pieces per row (40)
    constexpr int kPieces = kTM * kU8 / kThreads;
    static_assert(kTM * kU8 % kThreads == 0, "every thread fetches the same number of pieces");
    u32x4 piece[kPieces];
    auto fetch_piece = [&](int tile, int i) {
        const int q = threadIdx.x + i * kThreads, row = q / kU8, col = q % kU8;
        int cand = tile * kTM + row;
        cand = cand < n_d ? cand : 0;   // rows past the end repeat candidate 0; their outputs are not stored
        piece[i] = col < kH / 8 ? *reinterpret_cast<const u32x4*>(v_s + (size_t)cand * kH + 8 * col)
                                : *reinterpret_cast<const u32x4*>(v_d + (size_t)cand * kE + 8 * (col - kH / 8));
    };
    auto park_piece = [&](int buf, int i) {
        const int q = threadIdx.x + i * kThreads;
        *reinterpret_cast<u32x4*>(&U[buf][(q / kU8) * kUs + 8 * (q % kU8)]) = piece[i];
    };
    int tile = blockIdx.x;   // (no more workgroups than tiles)
#pragma unroll
    for (int i = 0; i < kPieces; ++i) fetch_piece(tile, i);
    bf16x8 whr[2][kU / 16];
    load_slices<kU / 16, kU / 16, u32x4>(whr, Wh, kU, wave, l32, half);
    static_assert(kThreads == kH, "one thread per hidden unit");
    cst[threadIdx.x] = bh[threadIdx.x];
    wo_lds[threadIdx.x] = wo[threadIdx.x];
#pragma unroll
    for (int i = 0; i < kPieces; ++i) park_piece(0, i);
#pragma unroll
    for (int i = 0; i < kPieces; ++i) fetch_piece(tile + (int)gridDim.x, i);
    __syncthreads();
    floatx16 bhr[2];
    bias_init(bhr, cst, wave, half);
    bf16x8 wof[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) wof[q] = last_layer_weights(wo_lds + 64 * wave, q, l32, half);
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
        for (int ks = 0; ks < kU / 16; ++ks) asm volatile("" : "+a"(whr[nt][ks]));

    floatx16 acc0[2], acc1[2], y0, y1;
    uint32_t pk[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) acc1[0][i] = acc1[1][i] = y0[i] = y1[i] = 0.f;
    auto store_rows = [&](int t, int buf) {   // a finished tile: the four wavefronts' shares of each row
        const int cand = t * kTM + (int)threadIdx.x;
        if (threadIdx.x < kTM && cand < n_d)
            y[cand] = (((red[buf][0][threadIdx.x] + red[buf][1][threadIdx.x]) + red[buf][2][threadIdx.x]) + red[buf][3][threadIdx.x]) + bo;
    };
    int buf = 0, done = 0;
    for (; tile < n_tiles; tile += gridDim.x, buf ^= 1, ++done) {
        // rows 0..31.  Meanwhile: the output of the previous tile's rows 32..63, the next tile's vectors to LDS.
        layer_from<kU / 16>(acc0, bhr, whr, U[buf], kUs, l32, half, [&](int i) {
            if (i < 8) {
                last_layer_pack(acc1, 2 * i, pk);
                last_layer_pack(acc1, 2 * i + 1, pk);
                if (i & 1) last_layer_mfma(y1, i >> 1, wof, pk);
            }
            if (i == 16 && half == 0) red[buf ^ 1][wave][32 + l32] = y1[0];
            if (i >= 20 && !(i & 1)) park_piece(buf ^ 1, (i - 20) >> 1);
        });
        static_assert(kPieces == 10 && kU / 16 == 20, "the ten pieces fit the layer's last twenty gaps");
        __syncthreads();   // the next tile's vectors and the previous tile's row outputs complete
        // rows 32..63.  Meanwhile: the output of rows 0..31, the requests for the tile after next, the previous tile's scores.
        layer_from<kU / 16>(acc1, bhr, whr, U[buf] + 32 * kUs, kUs, l32, half, [&](int i) {
            if (i < 8) {
                last_layer_pack(acc0, 2 * i, pk);
                last_layer_pack(acc0, 2 * i + 1, pk);
                if (i & 1) last_layer_mfma(y0, i >> 1, wof, pk);
            }
            if (i >= 8 && i < 8 + kPieces) fetch_piece(tile + 2 * (int)gridDim.x, i - 8);
            if (i == 20 && half == 0) red[buf][wave][l32] = y0[0];
            if (i == 24 && done > 0) store_rows(tile - (int)gridDim.x, buf ^ 1);
        });
        __syncthreads();   // this tile's buffer may be written again
    }
    // the last tile's rows 32..63
#pragma unroll
    for (int pair = 0; pair < 16; ++pair) last_layer_pack(acc1, pair, pk);
#pragma unroll
    for (int q = 0; q < 4; ++q) last_layer_mfma(y1, q, wof, pk);
    if (half == 0) red[buf ^ 1][wave][32 + l32] = y1[0];
    __syncthreads();
    store_rows(tile - (int)gridDim.x, buf ^ 1);
}

}  // namespace

size_t pacm_workspace_bytes(int64_t n_d)
{
    if (n_d < 0) n_d = 0;
    return round_up((size_t)n_d * kH * sizeof(float), 256) + round_up((size_t)n_d * kE * sizeof(float), 256);
}

}  // namespace pruner

using namespace pruner;

extern "C" int pruner_pacm_score(const float* feat, const int32_t* n_stmt, const float* flow, const int32_t* n_blk, int64_t n_d,
                                 const pruner_pacm* w, float* y, void* workspace, size_t workspace_bytes, void* stream)
{
    if (!feat || !n_stmt || !flow || !n_blk || !w || !y || n_d < 0 || n_d > (int64_t)(0x7FFFFFFF / (kS * kF))) return PRUNER_EINVAL;
    if (!w->W1 || !w->b1 || !w->W2 || !w->b2 || !w->We || !w->be || !w->Wq || !w->Wk || !w->Wv || !w->Wo || !w->Wh || !w->bh || !w->wo)
        return PRUNER_EINVAL;
    if (!aligned(feat, 16) || !aligned(flow, 4) || !aligned(n_stmt, 4) || !aligned(n_blk, 4) || !aligned(y, 4) || !aligned(w->W1, 8) ||
        !aligned(w->W2, 16) || !aligned(w->Wh, 16) || !aligned(w->b1, 4) || !aligned(w->b2, 4) || !aligned(w->be, 4) || !aligned(w->bh, 4) ||
        !aligned(w->We, 2) || !aligned(w->Wq, 2) || !aligned(w->Wk, 2) || !aligned(w->Wv, 2) || !aligned(w->Wo, 2) || !aligned(w->wo, 2))
        return PRUNER_EINVAL;
    if (!workspace || !aligned(workspace, 256)) return PRUNER_EWORKSPACE;
    if (workspace_bytes < pacm_workspace_bytes(n_d)) return PRUNER_EWORKSPACE;
    if (n_d == 0) return PRUNER_OK;
    int pacm_cus = 0;
    const int dev = current_device(&pacm_cus);
    if (dev < 0) return PRUNER_EHIP;
    hipStream_t st = static_cast<hipStream_t>(stream);
    char* ws = static_cast<char*>(workspace);
    uint16_t* v_s = reinterpret_cast<uint16_t*>(ws);
    uint16_t* v_d = reinterpret_cast<uint16_t*>(ws + round_up((size_t)n_d * kH * sizeof(uint16_t), 256));
    const int32_t n = (int32_t)n_d;
    // statement branch: one launch per kLocalCap x (compute units) candidates, groups as in pruner_verify_score
    const int64_t per_launch = (int64_t)kLocalCap * pacm_cus;
    for (int64_t c0 = 0; c0 < n_d; c0 += per_launch) {
        const int64_t m = n_d - c0 < per_launch ? n_d - c0 : per_launch;
        const int64_t grid = (m + kGroupMin - 1) / kGroupMin < pacm_cus ? (m + kGroupMin - 1) / kGroupMin : pacm_cus;
        int group_log = 3;
        while ((1 << group_log) < kGroupMax && m / (2 << group_log) >= 8 * grid) ++group_log;
        hipLaunchKernelGGL(pacm_stmt_kernel, dim3((unsigned)grid), dim3(kThreads), 0, st, feat + (size_t)c0 * kS * kF, n_stmt + c0, (int32_t)m, group_log,
                           w->W1, w->b1, w->W2, w->b2, v_s + (size_t)c0 * kH);
        PRUNER_LAUNCH_CHECK();
    }
    const int64_t head_tiles = (n_d + kTM - 1) / kTM;
    const int64_t flow_room = (int64_t)kFlowBlocksPerCu * pacm_cus;
    const int64_t flow_launch = (int64_t)kFlowLocalCap * kFlowWaves * flow_room;
    for (int64_t c0 = 0; c0 < n_d; c0 += flow_launch) {
        const int64_t m = n_d - c0 < flow_launch ? n_d - c0 : flow_launch;
        const int64_t blocks = (m + kFlowGroup * kFlowWaves - 1) / (kFlowGroup * kFlowWaves);
        hipLaunchKernelGGL(pacm_flow_kernel, dim3((unsigned)(blocks < flow_room ? blocks : flow_room)), dim3(kFlowThreads), 0, st,
                           flow + (size_t)c0 * kT * kD, n_blk + c0, (int32_t)m, w->We, w->be, w->Wq, w->Wk, w->Wv, w->Wo, v_d + (size_t)c0 * kE);
        PRUNER_LAUNCH_CHECK();
    }
    hipLaunchKernelGGL(pacm_head_kernel, dim3((unsigned)(head_tiles < pacm_cus ? head_tiles : pacm_cus)), dim3(kThreads), 0, st, v_s, v_d, n,
                       w->Wh, w->bh, w->wo, w->bo, y);
    PRUNER_LAUNCH_CHECK();
    return PRUNER_OK;
}
