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
// One launch for a set of at most 64 candidates per compute unit (pacm_small_kernel), three for larger ones:
//   pacm_stmt_kernel   the two statement layers on the matrix cores, tiles of 64 valid rows that hold whole candidates;
//                      a wavefront owns 64 hidden units and keeps its W1/W2 slices in registers
//   pacm_flow_kernel   the dataflow branch, a wavefront per tile of 32 block slots in quads, the chain from the features to
//                      the pooled vector in registers but for V
//   pacm_head_kernel   the head's hidden layer on the matrix cores (64 candidates per tile) and its output dot product
// The pooled vectors travel through the workspace (in one launch: through LDS) as the bfloat16 operands that the head's layer takes.
//
// A score is a function of its candidate alone: the same bits wherever in a set it stands and whatever stands beside it.  A
// matrix product of depth 16 adds its products in two groups of eight, one after the other (inside a group the order does not
// matter), so every product here has a candidate's own row or column to itself, and sums over rows run in a fixed order of
// the candidate's slots.
//
// Measured, before = eight padded slots per candidate in either branch and binary32 pooled vectors, the same bits (statement
// counts 3..8, blocks 0..5): 131,072 candidates: statement kernel 345 -> 196 us, dataflow 170 -> 66, head 43 -> 28, the call
// 518 -> 288; 8,192 candidates: 29.8 -> 19.3, 23.7 -> 9.8, 10.7 -> 9.5, the call 60 -> 37, in one launch 28.  (With the sums over rows on the matrix
// cores too, by the rows' places in a tile, 252 and 37: one score in a thousand then changed with the neighbours.)
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

__device__ __forceinline__ uint32_t bf16x2_of(float a, float b) { return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{a, b}), bf16x2)); }
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

// ---- statement branch ------------------------------------------------------------------------------------------------
// Tiles of 64 valid rows: a tile takes as many whole candidates as fit (at most 32), so the rows beyond n_stmt cost nothing, and
// a candidate never straddles.  The candidates of a workgroup are groups of neighbours, interleaved over the workgroups as
// in verify_mlp.hip; so are the weights in registers and the two halves of a tile half a layer apart.
// The sum over a candidate's rows is ((r0 + r1) + (r2 + r3)) + ((r4 + r5) + (r6 + r7)) in binary32, missing rows 0, wherever in
// a tile the rows lie: a score is a function of its candidate alone.  (Sums on the matrix cores, against a 0/1 matrix, add the
// rows in groups of eight by their place in the tile, and a pooled vector then depends on the neighbours.)  A wavefront parks
// the second hidden layer of its 64 units in LDS and reads the rows back candidate by candidate.
// Bound: what a SIMD's one wavefront issues in turn and waits for.  131,072 candidates, by the counters: the matrix pipe busy 36 %
// of the time, the vector ALU 29 %, LDS 35 %; weights and first rows on their way for small sets.

constexpr int kRowThreads = 8;                                   // threads that share a feature row: 128 contiguous bytes per request
constexpr int kXPass = kTM / (kThreads / kRowThreads);           // passes over the tile's rows (2)
constexpr int kXCols = (kF4 + kRowThreads - 1) / kRowThreads;    // float4 a thread fetches per row (6)
constexpr int kXLoads = kXPass * kXCols;                         // float4 a thread fetches per tile (12)
constexpr int kLocalCap = 2048;                                  // most candidates one workgroup takes in a launch
constexpr int kGroupMinLog = 3, kGroupMin = 1 << kGroupMinLog, kGroupMax = 64;   // neighbouring candidates that go to one workgroup together

// The candidates of a workgroup: groups first, first + stride, ... of 2^log neighbours.
struct Share {
    int log, first, stride, n_local;
    __device__ __forceinline__ Share(int n_d, int group_log, int my_first, int group_stride) : log(group_log), first(my_first), stride(group_stride)
    {
        const int n_groups = (n_d + (1 << log) - 1) >> log, my_groups = first < n_groups ? (n_groups - first + stride - 1) / stride : 0;
        const bool owns_last = my_groups > 0 && first + (my_groups - 1) * stride == n_groups - 1;
        n_local = (my_groups << log) - (owns_last ? (n_groups << log) - n_d : 0);
    }
    __device__ __forceinline__ int global_of(int l) const { return (((l >> log) * stride + first) << log) + (l & ((1 << log) - 1)); }
};

// The statement branch's places in LDS.
struct StmtLds {
    __bf16* arena;           // [kArena]
    float (*cst)[kH];        // [2]
    uint16_t* before;        // [candidates + 64 + 2]: valid rows of this workgroup's candidates 0..l-1 (at most 8 x kLocalCap)
    int32_t* row_src;        // [kTM]: what the rows of one tile are: candidate * 8 + statement, or -1
    uint32_t* scan_tot;      // [4]
};
constexpr int kArena = kTM * kXs + 2 * kTM * kHs + kHs;

struct StmtWeights {
    bf16x8 w1[2][kK1 / 16], w2[2][kH / 16];
    __device__ __forceinline__ void load_first(const uint16_t* __restrict__ W1, int wave, int l32, int half)
    {
        // W1's rows end at depth 164, the last step is four entries for half 0 and zeros otherwise
        static_assert(kK1 / 16 == kF / 16 + 1 && kF % 16 == 4, "W1's last depth step holds four entries");
        typedef u32x4 u32x4_a8 __attribute__((aligned(8)));   // W1's rows are 328 bytes
        load_slices<kK1 / 16, kF / 16, u32x4_a8>(w1, W1, kF, wave, l32, half);
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            const u32x2 tail = *reinterpret_cast<const u32x2*>(W1 + (size_t)(64 * wave + 32 * nt + l32) * kF + 16 * (kF / 16));
            u32x4 last = {0u, 0u, 0u, 0u};
            last[0] = half == 0 ? tail[0] : 0u;
            last[1] = half == 0 ? tail[1] : 0u;
            w1[nt][kF / 16] = __builtin_bit_cast(bf16x8, last);
        }
    }
    __device__ __forceinline__ void load_second(const uint16_t* __restrict__ W2, int wave, int l32, int half)
    {
        load_slices<kH / 16, kH / 16, u32x4>(w2, W2, kH, wave, l32, half);
    }
};

// Where the pooled statement vectors go: the workspace, or the head's operands in LDS (a row more than a tile's takes what
// is not to be stored).
struct PooledToMemory {
    static constexpr uint32_t kNowhere = 0xFFFF0000u;   // past the end of the buffer: no store
    __amdgpu_buffer_rsrc_t out;
    __device__ __forceinline__ PooledToMemory(uint16_t* v_s, int n_d) : out(__builtin_amdgcn_make_buffer_rsrc(v_s, 0, n_d * kH * 2, 0x00027000)) {}
    __device__ __forceinline__ uint32_t place(int cand, int local) const { return 2u * (uint32_t)cand * (uint32_t)kH; }
    __device__ __forceinline__ void store(u32x2 o, uint32_t to) const { __builtin_amdgcn_raw_buffer_store_b64(o, out, (int)to, 0, 0); }
};
struct PooledToLds {
    static constexpr uint32_t kNowhere = 2u * kTM * kUs;
    __bf16* U;
    __device__ __forceinline__ uint32_t place(int cand, int local) const { return 2u * (uint32_t)local * (uint32_t)kUs; }
    __device__ __forceinline__ void store(u32x2 o, uint32_t to) const { *reinterpret_cast<u32x2*>(reinterpret_cast<char*>(U) + to) = o; }
};

// between: other work of the workgroup, done (TOGETHER) while the first tile's features are on their way; it may use the arena.
template <bool TOGETHER, typename Out, typename Between>
__device__ __forceinline__ void stmt_branch(const StmtLds lds, const Share& share, const float* __restrict__ feat, const int32_t* __restrict__ n_stmt,
                                            const uint16_t* __restrict__ W1, const float* __restrict__ b1, const uint16_t* __restrict__ W2,
                                            const float* __restrict__ b2, const Out& out, Between&& between)
{
    __bf16* const X = lds.arena;               // feature tile, bfloat16 [kTM][kXs]
    __bf16* const H1 = lds.arena + kTM * kXs;  // first hidden layer of the tile [kTM][kHs]
    __bf16* const H2 = H1 + kTM * kHs;         // second hidden layer, and a row of zeros [kTM + 1][kHs]; a wavefront's 64 units are its own
    float(*const cst)[kH] = lds.cst;
    uint16_t* const before = lds.before;
    int32_t* const row_src = lds.row_src;
    uint32_t* const scan_tot = lds.scan_tot;
    StmtWeights weights;
    auto& w1r = weights.w1;
    auto& w2r = weights.w2;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int half = lane >> 5, l32 = lane & 31;
    const int n_local = share.n_local;
    auto global_of = [&](int l) -> int { return share.global_of(l); };

    // (the statement counts of the first candidates and the biases before the matrices, as in verify_mlp.hip: 8,192 candidates, this kernel
    // and the next, 30.8 -> 29.5 us)
    const int first_count = (int)threadIdx.x < n_local ? n_stmt[global_of((int)threadIdx.x)] : 0;
    const float b1_mine = b1[threadIdx.x], b2_mine = b2[threadIdx.x];
    __builtin_amdgcn_sched_barrier(0);
    weights.load_first(W1, wave, l32, half);
    static_assert(kThreads == kH, "one thread per hidden unit");
    cst[0][threadIdx.x] = b1_mine;
    cst[1][threadIdx.x] = b2_mine;

    {   // row numbering: exclusive scan of the statement counts, a run of `per` candidates per thread
        for (int l = threadIdx.x; l < n_local; l += kThreads) before[l] = (uint16_t)clamp8(l == (int)threadIdx.x ? first_count : n_stmt[global_of(l)]);
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
    auto tile_at = [&](int start) {
        Tile t;
        t.start = start;
        const int i = start + l32 < n_local ? start + l32 : n_local;
        const uint32_t b0 = before[i], b1v = before[i + 1];
        const uint32_t base = (uint32_t)__builtin_amdgcn_readfirstlane((int)b0);
        t.first = b0 - base;
        t.end = b1v - base;
        const bool in = start + l32 < n_local && t.end <= (uint32_t)kTM;
        t.count = (int)__popcll(__ballot(in) & 0xFFFFFFFFull);   // (the counts grow, so the candidates that fit are the first ones)
        t.cand = in ? global_of(start + l32) : -1;
        t.first = in ? t.first : 0u;
        t.end = in ? t.end : 0u;
        return t;
    };
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

    auto settle = [&]() {
        // the second layer's matrix: not needed before the first tile's second layer
        weights.load_second(W2, wave, l32, half);
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)   // weights in the accumulation registers (see verify_mlp.hip)
#pragma unroll
            for (int ks = 0; ks < kK1 / 16; ++ks) asm volatile("" : "+a"(w1r[nt][ks]));
        // the zero padding of the feature tile (depth 164..183) is written once
        for (int q = threadIdx.x; q < kTM * ((kXs - kF) / 4); q += kThreads) {
            const int r = q / ((kXs - kF) / 4), j = q % ((kXs - kF) / 4);
            *reinterpret_cast<uint2*>(&X[r * kXs + kF + 4 * j]) = make_uint2(0, 0);
        }
        for (int i = threadIdx.x; i < kHs; i += kThreads) H2[kTM * kHs + i] = (__bf16)0.f;
    };
    if constexpr (!TOGETHER) settle();

    floatx16 acc0[2], acc1[2];   // rows 0..31 and 32..63

    // The sums over the rows of the tile before, four candidates at a time: lanes 16 g .. 16 g + 15 take the g-th of them and
    // four hidden units each.  The first twelve candidates' (a tile of 64 rows holds 11.6 of five and a half rows) run in the
    // gaps between the MFMAs of two layers, a piece per gap and without a branch (one a gap cost 17 of 300 us at 131,072
    // candidates); a tile of more candidates goes through the others behind them.
    uint32_t pool_rows = 0, pool_to = Out::kNowhere;   // the l32-th candidate: first row, number of rows << 8; where its sums go
    int pool_count = 0;
    const int p_group = lane >> 4, p_unit = 64 * wave + 4 * (lane & 15);
    uint32_t p_n = 0, p_to = 0;
    const __bf16* p_from = H2;
    u32x2 p_raw[kS];
    f32x4 p_sum[4];
    constexpr int kPoolPieces = 13;
    auto pool_piece = [&](int first, int piece) {   // candidates first .. first + 3 of the tile
        if (piece == 0) {
            const uint32_t rows = (uint32_t)__shfl((int)pool_rows, first + p_group, 64);
            p_to = (uint32_t)__shfl((int)pool_to, first + p_group, 64) + 2u * (uint32_t)p_unit;
            p_n = rows >> 8;
            p_from = H2 + (rows & 0xFFu) * kHs + p_unit;
        }
        if (piece == 1 || piece == 2) {
#pragma unroll
            for (int r = 4 * (piece - 1); r < 4 * piece; ++r)
                p_raw[r] = *reinterpret_cast<const u32x2*>((uint32_t)r < p_n ? p_from + r * kHs : H2 + kTM * kHs + p_unit);
        }
        if (piece >= 3 && piece < 11) {   // rows 2 q and 2 q + 1, two units
            const int q = (piece - 3) >> 1, w = (piece - 3) & 1;
            p_sum[q][2 * w] = __uint_as_float(p_raw[2 * q][w] << 16) + __uint_as_float(p_raw[2 * q + 1][w] << 16);
            p_sum[q][2 * w + 1] = __uint_as_float(p_raw[2 * q][w] & 0xFFFF0000u) + __uint_as_float(p_raw[2 * q + 1][w] & 0xFFFF0000u);
        }
        if (piece == 11) {
#pragma unroll
            for (int q = 0; q < 4; q += 2)
#pragma unroll
                for (int e = 0; e < 4; ++e) p_sum[q][e] += p_sum[q + 1][e];
        }
        if (piece == 12) {
#pragma unroll
            for (int e = 0; e < 4; ++e) p_sum[0][e] += p_sum[2][e];
            const u32x2 o = {bf16x2_of(p_sum[0][0], p_sum[0][1]), bf16x2_of(p_sum[0][2], p_sum[0][3])};
            out.store(o, p_to);
        }
    };
    constexpr int kPoolAhead = 12, kPoolGaps = 2 * (kK1 / 16 + kH / 16) / (kPoolAhead / 4);   // gaps per four candidates (18)
    static_assert(kPoolGaps >= kPoolPieces, "a piece per gap");
    auto pool_gap = [&](int gap) {   // (a constant after unrolling) the pieces spread evenly over the gaps
        const int at = gap % kPoolGaps, piece = (at * kPoolPieces + kPoolGaps - 1) / kPoolGaps;
        if (gap < kPoolAhead / 4 * kPoolGaps && piece < kPoolPieces && piece * kPoolGaps / kPoolPieces == at) pool_piece(4 * (gap / kPoolGaps), piece);
    };
    auto pool_rest = [&](int first) {
        for (; first < pool_count; first += 4) {
#pragma unroll
            for (int piece = 0; piece < kPoolPieces; ++piece) pool_piece(first, piece);
        }
    };

#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc1[nt][i] = 0.f;
    Tile cur = tile_at(0);
    if (wave == 0) write_rows(cur);
    __syncthreads();
    fetch_read();
#pragma unroll
    for (int i = 0; i < kXLoads; ++i) fetch_issue(i);
    Tile nxt = tile_at(cur.start + cur.count);
    if constexpr (TOGETHER) {
        __builtin_amdgcn_sched_barrier(0);
        between();
    }
    __syncthreads();   // everyone has read the first tile's rows
    if constexpr (TOGETHER) settle();
    if (wave == 0) write_rows(nxt);
#pragma unroll
    for (int i = 0; i < kXLoads; ++i) park_piece(i);
    bias_init(acc0, cst[0], wave, half);
    __syncthreads();
    fetch_read();
#pragma unroll
    for (int i = 0; i < kXLoads; ++i) fetch_issue(i);

    // A tile in four stages, each a layer of one half of the rows with other work between its MFMAs.  At the loop's head
    // X holds this tile's rows and the next tile's are on their way to registers.
    while (cur.count > 0) {
        // layer 1, rows 0..31.  Meanwhile: the previous tile's second hidden layer of rows 32..63 to LDS.
        layer<kK1 / 16>(acc0, w1r, X, kXs, l32, half, [&](int i) {
            if (i < 16 && !(i & 1)) park_hidden(acc1, i >> 1, H2 + 32 * kHs, kHs, wave, l32, half);
            if (i == 18) bias_init(acc1, cst[0], wave, half);
            if (i == 20) wave_lds_fence();
        });
        // layer 1, rows 32..63.  Meanwhile: hidden layer 1 of rows 0..31 to LDS, sums over the previous tile's rows.
        layer<kK1 / 16>(acc1, w1r, X + 32 * kXs, kXs, l32, half, [&](int i) {
            pool_gap(i);
            if (i >= 4 && i < 20 && !(i & 1)) park_hidden(acc0, (i - 4) >> 1, H1, kHs, wave, l32, half);
            if (i == 20) bias_init(acc0, cst[1], wave, half);
        });
        __syncthreads();   // rows 0..31 of H1 complete; X no longer read
        // layer 2, rows 0..31.  Meanwhile: hidden layer 1 of rows 32..63 and the next tile's features to LDS, more of the sums, and
        // what the rows of the tile after next are.
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)   // (no instruction: the register class, and in the first tile the wait for the matrix)
            asm volatile("" : "+a"(w2r[nt][0]), "+a"(w2r[nt][1]), "+a"(w2r[nt][2]), "+a"(w2r[nt][3]), "+a"(w2r[nt][4]), "+a"(w2r[nt][5]),
                              "+a"(w2r[nt][6]), "+a"(w2r[nt][7]), "+a"(w2r[nt][8]), "+a"(w2r[nt][9]), "+a"(w2r[nt][10]), "+a"(w2r[nt][11]),
                              "+a"(w2r[nt][12]), "+a"(w2r[nt][13]), "+a"(w2r[nt][14]), "+a"(w2r[nt][15]));
        static_assert(kH / 16 == 16, "the second layer's sixteen depth steps are listed above");
        Tile after = nxt;
        layer<kH / 16>(acc0, w2r, H1, kHs, l32, half, [&](int i) {
            pool_gap(2 * (kK1 / 16) + i);
            if (i & 1) {
                if (i >= 2 * (kH / 16 - kXLoads)) park_piece((i - 2 * (kH / 16 - kXLoads)) >> 1);   // as late as the layer allows
                return;
            }
            if (i < 16) park_hidden(acc1, i >> 1, H1 + 32 * kHs, kHs, wave, l32, half);
            if (i == 18) after = tile_at(nxt.start + nxt.count);
            if (i == 20) bias_init(acc1, cst[1], wave, half);
            if (i == 26 && wave == 0) write_rows(after);
        });
        pool_rest(kPoolAhead);
        pool_count = cur.count;
        pool_rows = cur.first | ((cur.end - cur.first) << 8);
        pool_to = cur.cand >= 0 ? out.place(cur.cand, cur.start + l32) : Out::kNowhere;
        wave_lds_fence();
        __syncthreads();   // rows 32..63 of H1, X (the next tile's rows) and the rows' table complete
        // layer 2, rows 32..63.  Meanwhile: the second hidden layer of rows 0..31 to LDS, and the requests for the rows of the
        // tile after next.
        layer<kH / 16>(acc1, w2r, H1 + 32 * kHs, kHs, l32, half, [&](int i) {
            if (!(i & 1) && i < 16) park_hidden(acc0, i >> 1, H2, kHs, wave, l32, half);
            if (i == 0) fetch_read();
            if ((i & 1) && i < 2 * kXLoads) fetch_issue(i >> 1);
            if (i == 26) bias_init(acc0, cst[0], wave, half);
        });
        cur = nxt;
        nxt = after;
    }
    // the last tile's second half
#pragma unroll
    for (int piece = 0; piece < 8; ++piece) park_hidden(acc1, piece, H2 + 32 * kHs, kHs, wave, l32, half);
    wave_lds_fence();
    pool_rest(0);
}

__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(1, 1)))
pacm_stmt_kernel(const float* __restrict__ feat, const int32_t* __restrict__ n_stmt, int32_t n_d, int group_log, const uint16_t* __restrict__ W1,
                 const float* __restrict__ b1, const uint16_t* __restrict__ W2, const float* __restrict__ b2, uint16_t* __restrict__ v_s)
{
    __shared__ __attribute__((aligned(16))) __bf16 arena[kArena];
    __shared__ __attribute__((aligned(16))) float cst[2][kH];
    __shared__ uint16_t before[kLocalCap + 64 + 2];
    __shared__ int32_t row_src[kTM];
    __shared__ uint32_t scan_tot[4];
    const Share share(n_d, group_log, (int)blockIdx.x, (int)gridDim.x);
    stmt_branch<false>(StmtLds{arena, cst, before, row_src, scan_tot}, share, feat, n_stmt, W1, b1, W2, b2, PooledToMemory(v_s, n_d), []() {});
}

// ---- dataflow branch -------------------------------------------------------------------------------------------------
// A wavefront works on tiles of 32 block slots, eight quads of four: a candidate of up to four blocks takes one quad, of more two
// neighbouring ones that begin at an even quad, one of none takes no slot.  The chain stays in registers: every layer is
// computed transposed (weights as the A operand), which leaves a lane 16 units of its row, and the rounded result is the
// operand of the next product once the two halves of the wavefront have exchanged half of it (half 0 then holds the lower eight
// of sixteen neighbouring units, as the weights do).  The scores come with a query per lane and the keys of one parity of
// quads per half: four of them are the query's.  Only V goes through LDS, from which a query's lane reads its candidate's rows.
// Every sum runs over a candidate's own slots in a fixed order, wherever in a tile they lie (softmax and pooled vectors ((0 + 1)
// + (2 + 3)) + ((4 + 5) + (6 + 7)), the products with the attention weights one key after the other): a score is a function of
// its candidate alone, and nothing of one candidate reaches another.
// Bound: vector instructions, and the waits between dependent stages (131,072 candidates, by the counters: vector ALU busy 74 %
// of the time where every candidate takes two quads, 47 % with 2.8 blocks on average and a third of the tiles).

constexpr int kFlowWaves = 4;                 // wavefronts per workgroup, each with tiles of its own
constexpr int kFlowThreads = 64 * kFlowWaves;
constexpr int kFlowGroupLog = 3, kFlowGroup = 1 << kFlowGroupLog;   // neighbouring candidates that go to one wavefront together
constexpr int kFlowRows = 32;
constexpr int kFlowQuads = kFlowRows / 4;
constexpr int kFlowBlocksPerCu = 2;
constexpr int kDk = 32;                       // 23 padded to the MFMA depth
constexpr int kVs = kE + 8;                   // LDS row stride of V (bfloat16 elements)
constexpr int kFlowLocalCap = 1024;           // most candidates of one wavefront in a launch

// Exchanges inside a group of eight neighbouring lanes at the vector ALU's own rate: CTRL 0xB1 brings the neighbour's value
// (lane ^ 1), 0x4E the other pair's (lane ^ 2), 0x141 mirrors the row half (lane 7 - j of the eight, i.e. the other quad).
template <int CTRL> __device__ __forceinline__ float across8(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ float sum4(float x)
{
    x += across8<0xB1>(x);
    x += across8<0x4E>(x);
    return x;
}

// Pairs of neighbouring units as a product leaves them (units 8 (p / 2) + 4 half + 2 (p % 2) and the next, p = 0..3) as an operand:
// units 8 half + 2 p and the next.
__device__ __forceinline__ bf16x8 operand_of(uint32_t p0, uint32_t p1, uint32_t p2, uint32_t p3)
{
    const auto a = __builtin_amdgcn_permlane32_swap(p0, p2, false, false), b = __builtin_amdgcn_permlane32_swap(p1, p3, false, false);
    return __builtin_bit_cast(bf16x8, u32x4{a[0], b[0], a[1], b[1]});
}
__device__ __forceinline__ bf16x8 plain_operand(const floatx16& a, int q)   // registers 8 q .. 8 q + 7
{
    return operand_of(bf16x2_of(a[8 * q], a[8 * q + 1]), bf16x2_of(a[8 * q + 2], a[8 * q + 3]), bf16x2_of(a[8 * q + 4], a[8 * q + 5]),
                      bf16x2_of(a[8 * q + 6], a[8 * q + 7]));
}

// LDS of the dataflow branch for CAP candidates per wavefront.
template <int CAP> struct FlowLds {
    uint8_t counts[kFlowWaves][CAP];                // blocks of the wavefront's candidates
    uint32_t quad_tab[kFlowWaves][2][kFlowQuads];   // what the quads of a tile are (two tiles are in the making)
    __attribute__((aligned(16))) u32x4 wv[2][kE / 16][64], wo[2][kE / 16][64];   // Wv's and Wo's fragments (registers hold the others)
    __attribute__((aligned(16))) __bf16 v[kFlowWaves][(kFlowRows + 1) * kVs];    // a tile's V, and a row of zeros
    __attribute__((aligned(16))) float be[kE];
};

// Weights as A operands, lane (l32, half): eight depths 16 ks + 8 half + j of row 32 nt + l32.
struct FlowWeights {
    bf16x8 e[2][kDk / 16], q[2][kE / 16], k[2][kE / 16];
    u32x4 staged[kE / 16];   // a quarter of Wo and Wv, on their way to LDS: wavefront w has block w / 2 of one of them
    float be;
    __device__ __forceinline__ void load(const uint16_t* __restrict__ We, const float* __restrict__ be_, const uint16_t* __restrict__ Wq,
                                         const uint16_t* __restrict__ Wk, const uint16_t* __restrict__ Wv, const uint16_t* __restrict__ Wo, int wave, int l32,
                                         int half)
    {
        be = be_[threadIdx.x & (kE - 1)];
        auto fragment = [&](const uint16_t* W, int n, int ks) {
            typedef u32x4 u32x4_a2 __attribute__((aligned(2)));
            return u32x4(*reinterpret_cast<const u32x4_a2*>(W + (size_t)n * kE + 16 * ks + 8 * half));
        };
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            const int n = 32 * nt + l32;
#pragma unroll
            for (int ks = 0; ks < kDk / 16; ++ks) {
                uint32_t pk[4];
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    const int k0 = 16 * ks + 8 * half + 2 * p;   // (depths past the last repeat it and are cleared)
                    const uint32_t lo = We[n * kD + (k0 < kD ? k0 : kD - 1)], hi = We[n * kD + (k0 + 1 < kD ? k0 + 1 : kD - 1)];
                    pk[p] = (k0 < kD ? lo : 0u) | (k0 + 1 < kD ? hi << 16 : 0u);
                }
                e[nt][ks] = __builtin_bit_cast(bf16x8, u32x4{pk[0], pk[1], pk[2], pk[3]});
            }
#pragma unroll
            for (int ks = 0; ks < kE / 16; ++ks) {
                q[nt][ks] = __builtin_bit_cast(bf16x8, fragment(Wq, n, ks));
                k[nt][ks] = __builtin_bit_cast(bf16x8, fragment(Wk, n, ks));
            }
        }
#pragma unroll
        for (int ks = 0; ks < kE / 16; ++ks) staged[ks] = fragment(wave & 1 ? Wv : Wo, 32 * (wave >> 1) + l32, ks);
        static_assert(kFlowWaves == 4, "two blocks of two matrices");
    }
};

// global_of: the wavefront's candidates 0 .. n_local - 1, the first of which have first_count blocks, one to a lane; dest: where the
// pooled vector of such a candidate goes (64 units).
template <int CAP, typename Global, typename Dest>
__device__ __forceinline__ void flow_branch(FlowLds<CAP>& lds, int n_local, Global&& global_of, Dest&& dest, const float* __restrict__ flow,
                                            const int32_t* __restrict__ n_blk, int first_count, const FlowWeights& weights)
{
    auto& wer = weights.e;
    auto& wqr = weights.q;
    auto& wkr = weights.k;
    auto& counts = lds.counts;
    auto& quad_tab = lds.quad_tab;
    auto& wv_lds = lds.wv;
    auto& wo_lds = lds.wo;
    auto& v_lds = lds.v;
    auto& be_lds = lds.be;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int half = lane >> 5, l32 = lane & 31;
#pragma unroll
    for (int ks = 0; ks < kE / 16; ++ks) (wave & 1 ? wv_lds : wo_lds)[wave >> 1][ks][lane] = weights.staged[ks];
    if (threadIdx.x < kE) be_lds[threadIdx.x] = weights.be;
    for (int l = lane; l < n_local; l += 64) counts[wave][l] = (uint8_t)clamp8(l == lane ? first_count : n_blk[global_of(l)]);
    __bf16* const V = v_lds[wave];
    for (int i = lane; i < kVs; i += 64) V[kFlowRows * kVs + i] = (__bf16)0.f;
    __syncthreads();   // (the only one: from here on every wavefront goes its own way)

    struct Tile {
        int start, count;
        uint32_t quad;         // of the lane's (l32-th) row: its candidate's first quad | blocks << 8 | place among the tile's candidates << 16
        f32x4 x[4];            // the lane's eight plus eight (half 1: eight) features of that row
    };
    auto zero16 = []() {
        floatx16 z;
#pragma unroll
        for (int i = 0; i < 16; ++i) z[i] = 0.f;
        return z;
    };
    // The tile from local candidate `start` on; its features are requested.
    auto tile_at = [&](int start, int buffer) {
        Tile t;
        t.start = start;
        const bool there = start + l32 < n_local;
        const uint32_t n = there ? counts[wave][start + l32] : 0u;
        // places: a candidate of two quads begins at an even one, so the parity before it is that of the candidates of one
        // quad since the last of two
        const uint32_t one = (uint32_t)__ballot(n >= 1u && n <= 4u), two = (uint32_t)__ballot(n > 4u), lower = (1u << l32) - 1u;
        const uint32_t behind = two & lower ? ~0u << (31 - __clz((int)(two & lower))) : ~0u;
        const uint32_t padded = (uint32_t)__ballot(n > 4u && (__popc(one & lower & behind) & 1)) & (lower | (1u << l32));
        const uint32_t first = (uint32_t)(__popc(one & lower) + 2 * __popc(two & lower) + __popc(padded)), quads = n == 0u ? 0u : n <= 4u ? 1u : 2u;
        const bool in = there && first + quads <= (uint32_t)kFlowQuads;
        t.count = (int)__popc((uint32_t)__ballot(in));   // (the places grow, so the candidates that fit are the first ones)
        uint32_t* tab = quad_tab[wave][buffer];
        if (lane < kFlowQuads) tab[lane] = 0u;
        wave_lds_fence();
        if (in && half == 0) {
            const uint32_t what = first | (n << 8) | ((uint32_t)l32 << 16);
            if (quads >= 1u) tab[first] = what;
            if (quads == 2u) tab[first + 1] = what;
        }
        if (in && quads == 0u) {   // no blocks: its vector is zero
            u32x4* to = reinterpret_cast<u32x4*>(dest(start + l32) + 32 * half);
#pragma unroll
            for (int i = 0; i < 4; ++i) to[i] = u32x4{0u, 0u, 0u, 0u};
        }
        wave_lds_fence();
        t.quad = tab[l32 >> 2];
        const uint32_t slot = (uint32_t)l32 - 4u * (t.quad & 0xFFu);
        const int64_t src = slot < ((t.quad >> 8) & 0xFFu) ? (int64_t)global_of(start + (int)(t.quad >> 16)) * kT + slot : 0;
        typedef f32x4 f32x4_a4 __attribute__((aligned(4)));
        const float* r = flow + src * kD;
        t.x[0] = *reinterpret_cast<const f32x4_a4*>(r + 8 * half);
        t.x[1] = *reinterpret_cast<const f32x4_a4*>(r + 8 * half + 4);
        t.x[2] = *reinterpret_cast<const f32x4_a4*>(r + (half ? 8 : 16));
        t.x[3] = *reinterpret_cast<const f32x4_a4*>(r + (half ? 8 : 19));   // depths 20, 21, 22 are its last three
        return t;
    };

    Tile cur = tile_at(0, 0);
    int buffer = 1;
    do {   // (a wavefront without candidates goes through it once and stores nothing)
        const Tile nxt = tile_at(cur.start + cur.count, buffer);
        buffer ^= 1;
        const int first_quad = (int)(cur.quad & 0xFFu), n_mine = (int)((cur.quad >> 8) & 0xFFu), slot = l32 - 4 * first_quad;
        const bool row_there = slot < n_mine;   // (a quad that is not taken has n_mine = 0)
        // features, bfloat16, depth 23..31 zero
        bf16x8 d[2];
        {
            const uint32_t there = row_there ? ~0u : 0u;
            const u32x4 d0 = {bf16x2_of(cur.x[0][0], cur.x[0][1]) & there, bf16x2_of(cur.x[0][2], cur.x[0][3]) & there,
                              bf16x2_of(cur.x[1][0], cur.x[1][1]) & there, bf16x2_of(cur.x[1][2], cur.x[1][3]) & there};
            const uint32_t low = half ? 0u : there;
            const u32x4 d1 = {bf16x2_of(cur.x[2][0], cur.x[2][1]) & low, bf16x2_of(cur.x[2][2], cur.x[2][3]) & low,
                              bf16x2_of(cur.x[3][1], cur.x[3][2]) & low, bf16x2_of(cur.x[3][3], 0.f) & low};
            d[0] = __builtin_bit_cast(bf16x8, d0);
            d[1] = __builtin_bit_cast(bf16x8, d1);
        }
        uint32_t e_pair[16];   // E as the product leaves it: pairs of units 32 nt + 8 (p / 2) + 4 half + 2 (p % 2), p = index - 8 nt
        bf16x8 e[kE / 16];     // ... and as an operand
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            floatx16 acc;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const f32x4 b = *reinterpret_cast<const f32x4*>(&be_lds[32 * nt + 8 * g + 4 * half]);
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[4 * g + j] = b[j];
            }
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wer[nt][0], d[0], acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wer[nt][1], d[1], acc, 0, 0, 0);
#pragma unroll
            for (int p = 0; p < 8; ++p) e_pair[8 * nt + p] = relu_bf16x2(acc[2 * p], acc[2 * p + 1]);
#pragma unroll
            for (int hq = 0; hq < 2; ++hq) {
                const int p = 8 * nt + 4 * hq;
                e[2 * nt + hq] = operand_of(e_pair[p], e_pair[p + 1], e_pair[p + 2], e_pair[p + 3]);
            }
        }
        floatx16 sc;
        {
            bf16x8 q[kE / 16], k[kE / 16];
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) {
                floatx16 aq = zero16(), ak = zero16(), av = zero16();
#pragma unroll
                for (int ks = 0; ks < kE / 16; ++ks) {
                    aq = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wqr[nt][ks], e[ks], aq, 0, 0, 0);
                    ak = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wkr[nt][ks], e[ks], ak, 0, 0, 0);
                    av = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wv_lds[nt][ks][lane]), e[ks], av, 0, 0, 0);
                }
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const u32x2 o = {bf16x2_of(av[4 * g], av[4 * g + 1]), bf16x2_of(av[4 * g + 2], av[4 * g + 3])};
                    *reinterpret_cast<u32x2*>(&V[l32 * kVs + 32 * nt + 8 * g + 4 * half]) = o;
                }
#pragma unroll
                for (int hq = 0; hq < 2; ++hq) {
                    q[2 * nt + hq] = plain_operand(aq, hq);
                    k[2 * nt + hq] = plain_operand(ak, hq);
                }
            }
            sc = zero16();
#pragma unroll
            for (int ks = 0; ks < kE / 16; ++ks) sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k[ks], q[ks], sc, 0, 0, 0);   // lane: query l32, keys 8 (i / 4) + 4 half + i % 4
        }
        wave_lds_fence();
        // Softmax.  Of the candidate's one or two quads of keys this half holds the one of its parity (four registers), the other
        // half the other.
        float weight[kT];   // of the candidate's keys in order; 0 past its last
        {
            const int mine = first_quad + ((first_quad ^ half) & 1), key0 = 4 * (mine - first_quad);
            const int left = n_mine - key0;   // of the quad's keys, those that are there
            float p[4], mx = -__builtin_inff();
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int b = mine >> 1;
                const float s = b == 0 ? sc[r] : b == 1 ? sc[4 + r] : b == 2 ? sc[8 + r] : sc[12 + r];
                p[r] = r < left ? s * 0.125f : -__builtin_inff();
                mx = fmaxf(mx, p[r]);
            }
            mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
#pragma unroll
            for (int r = 0; r < 4; ++r) p[r] = r < left ? expf(p[r] - mx) : 0.f;
            float den = (p[0] + p[1]) + (p[2] + p[3]);
            den += __shfl_xor(den, 32, 64);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float w = n_mine > 0 ? p[r] / den : 0.f, other = __shfl_xor(w, 32, 64);
                weight[r] = key0 == 0 ? w : other;
                weight[4 + r] = key0 == 0 ? other : w;
            }
        }
        // o = sum over the keys of weight v in binary32, one key after the other; the lane has its query's units 16 ks + 8 half ..
        bf16x8 o[kE / 16];
        {
            float acc[kE / 16][8];
#pragma unroll
            for (int ks = 0; ks < kE / 16; ++ks)
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[ks][j] = 0.f;
            const bool two_quads = __ballot(n_mine > 4) != 0ull;
            const __bf16* const own = V + (4 * first_quad) * kVs + 8 * half;
            const __bf16* const none = V + kFlowRows * kVs + 8 * half;
            auto add_keys = [&](int from) {
#pragma unroll
                for (int j = from; j < from + 4; ++j) {
                    const __bf16* row = j < n_mine ? own + j * kVs : none;
#pragma unroll
                    for (int ks = 0; ks < kE / 16; ++ks) {
                        const u32x4 v = *reinterpret_cast<const u32x4*>(row + 16 * ks);
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            acc[ks][2 * c] = __builtin_fmaf(weight[j], __uint_as_float(v[c] << 16), acc[ks][2 * c]);
                            acc[ks][2 * c + 1] = __builtin_fmaf(weight[j], __uint_as_float(v[c] & 0xFFFF0000u), acc[ks][2 * c + 1]);
                        }
                    }
                }
            };
            add_keys(0);
            if (two_quads) add_keys(4);
#pragma unroll
            for (int ks = 0; ks < kE / 16; ++ks) {
                const u32x4 f = {bf16x2_of(acc[ks][0], acc[ks][1]), bf16x2_of(acc[ks][2], acc[ks][3]), bf16x2_of(acc[ks][4], acc[ks][5]),
                                 bf16x2_of(acc[ks][6], acc[ks][7])};
                o[ks] = __builtin_bit_cast(bf16x8, f);
            }
        }
        // z = e + Wo o, summed over the candidate's blocks: every lane of its quads then holds the sums, and lane j of the first
        // quad stores the units 32 nt + 8 j + 4 half ..
        const bool stores = n_mine > 0 && (l32 >> 2) == first_quad;
        uint16_t* const to = dest(stores ? cur.start + (int)(cur.quad >> 16) : 0) + 8 * (l32 & 3) + 4 * half;
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            floatx16 z = zero16();
#pragma unroll
            for (int ks = 0; ks < kE / 16; ++ks) z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wo_lds[nt][ks][lane]), o[ks], z, 0, 0, 0);
            f32x4 run = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const uint32_t pair = e_pair[8 * nt + i / 2];
                const float e_res = __uint_as_float(i & 1 ? pair & 0xFFFF0000u : pair << 16);
                float sum = sum4(row_there ? e_res + z[i] : 0.f);
                const float both = sum + across8<0x141>(sum);
                sum = n_mine > 4 ? both : sum;
                run[i & 3] = (l32 & 3) == i / 4 ? sum : run[i & 3];
            }
            if (stores) *reinterpret_cast<u32x2*>(to + 32 * nt) = u32x2{bf16x2_of(run[0], run[1]), bf16x2_of(run[2], run[3])};
        }
        cur = nxt;
    } while (cur.count > 0);
}

__global__ void __launch_bounds__(kFlowThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
pacm_flow_kernel(const float* __restrict__ flow, const int32_t* __restrict__ n_blk, int32_t n_d, const uint16_t* __restrict__ We,
                 const float* __restrict__ be, const uint16_t* __restrict__ Wq, const uint16_t* __restrict__ Wk,
                 const uint16_t* __restrict__ Wv, const uint16_t* __restrict__ Wo, uint16_t* __restrict__ v_d)
{
    __shared__ FlowLds<kFlowLocalCap> lds;
    const Share share(n_d, kFlowGroupLog, (int)blockIdx.x * kFlowWaves + (int)(threadIdx.x >> 6), (int)gridDim.x * kFlowWaves);   // this wavefront's candidates
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int first_count = lane < share.n_local ? n_blk[share.global_of(lane)] : 0;   // (on its way with the weights)
    __builtin_amdgcn_sched_barrier(0);
    FlowWeights weights;
    weights.load(We, be, Wq, Wk, Wv, Wo, wave, lane & 31, lane >> 5);
    flow_branch(lds, share.n_local, [&](int l) { return share.global_of(l); }, [&](int l) { return v_d + (size_t)share.global_of(l) * kE; }, flow, n_blk,
                first_count, weights);
}

// ---- head ------------------------------------------------------------------------------------------------------------
// The two 32-row halves of a tile run one after the other on the matrix cores; rounding, the output dot product (binary32, in
// the order of a lane's units) and the stores of one half, and the next tile's way into LDS, are issued between the MFMAs
// of the other.  Two tiles' operands in LDS, two barriers per tile.  131,072 candidates: 640 bytes each at 3 TB/s, matrix pipe
// busy 26 % of the time, vector ALU 20 %; weights and launch for small sets.

__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(1, 1)))
pacm_head_kernel(const uint16_t* __restrict__ v_s, const uint16_t* __restrict__ v_d, int32_t n_d, const uint16_t* __restrict__ Wh,
                 const float* __restrict__ bh, const uint16_t* __restrict__ wo, float bo, float* __restrict__ y)
{
    __shared__ __attribute__((aligned(16))) __bf16 U[2][kTM * kUs];   // a tile's concatenated pooled vectors
    __shared__ __attribute__((aligned(16))) float cst[kH];
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
    cst[threadIdx.x] = bh[threadIdx.x];
    float wor[2][16];   // this lane's output weights, in accumulator order
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
        for (int i = 0; i < 16; ++i) wor[nt][i] = __uint_as_float((uint32_t)wo[64 * wave + 32 * nt + 8 * (i / 4) + 4 * half + (i % 4)] << 16);
#pragma unroll
    for (int i = 0; i < kPieces; ++i) park_piece(0, i);
#pragma unroll
    for (int i = 0; i < kPieces; ++i) fetch_piece(tile + (int)gridDim.x, i);
    __syncthreads();
    floatx16 bhr[2];
    bias_init(bhr, cst, wave, half);
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
        for (int ks = 0; ks < kU / 16; ++ks) asm volatile("" : "+a"(whr[nt][ks]));

    floatx16 acc0[2], acc1[2];
    float part = 0.f;
    // the output of a half's rows, pair by pair of a lane's units
    auto dot_pair = [&](const floatx16(&acc)[2], int pair) {
        const int nt = pair >> 3, p = pair & 7;
        const uint32_t pr = relu_bf16x2(acc[nt][2 * p], acc[nt][2 * p + 1]);
        part = __builtin_fmaf(__uint_as_float(pr << 16), wor[nt][2 * p], pair == 0 ? 0.f : part);
        part = __builtin_fmaf(__uint_as_float(pr & 0xFFFF0000u), wor[nt][2 * p + 1], part);
    };
    auto dot_park = [&](int buf, int hh) {
        part += __shfl_xor(part, 32, 64);
        if (half == 0) red[buf][wave][32 * hh + l32] = part;
    };
#pragma unroll
    for (int i = 0; i < 16; ++i) acc1[0][i] = acc1[1][i] = 0.f;
    auto store_rows = [&](int t, int buf) {   // a finished tile: the four wavefronts' shares of each row
        const int cand = t * kTM + (int)threadIdx.x;
        if (threadIdx.x < kTM && cand < n_d)
            y[cand] = (((red[buf][0][threadIdx.x] + red[buf][1][threadIdx.x]) + red[buf][2][threadIdx.x]) + red[buf][3][threadIdx.x]) + bo;
    };
    int buf = 0, done = 0;
    for (; tile < n_tiles; tile += gridDim.x, buf ^= 1, ++done) {
        // rows 0..31.  Meanwhile: the output of the previous tile's rows 32..63, the next tile's vectors to LDS.
        layer_from<kU / 16>(acc0, bhr, whr, U[buf], kUs, l32, half, [&](int i) {
            if (i < 16) dot_pair(acc1, i);
            if (i == 16) dot_park(buf ^ 1, 1);
            if (i >= 20 && !(i & 1)) park_piece(buf ^ 1, (i - 20) >> 1);
        });
        static_assert(kPieces == 10 && kU / 16 == 20, "the ten pieces fit the layer's last twenty gaps");
        __syncthreads();   // the next tile's vectors and the previous tile's row outputs complete
        // rows 32..63.  Meanwhile: the output of rows 0..31, the requests for the tile after next, the previous tile's scores.
        layer_from<kU / 16>(acc1, bhr, whr, U[buf] + 32 * kUs, kUs, l32, half, [&](int i) {
            if (i < 16) dot_pair(acc0, i);
            if (i >= 8 && i < 8 + kPieces) fetch_piece(tile + 2 * (int)gridDim.x, i - 8);
            if (i == 20) dot_park(buf, 0);
            if (i == 24 && done > 0) store_rows(tile - (int)gridDim.x, buf ^ 1);
        });
        __syncthreads();   // this tile's buffer may be written again
    }
    // the last tile's rows 32..63
#pragma unroll
    for (int pair = 0; pair < 16; ++pair) dot_pair(acc1, pair);
    dot_park(buf ^ 1, 1);
    __syncthreads();
    store_rows(tile - (int)gridDim.x, buf ^ 1);
}

// ---- all three in one launch -----------------------------------------------------------------------------------------
// Small sets: a workgroup takes its candidates (one tile of the head at most) through both branches and the head, the pooled
// vectors staying in LDS.  The dataflow branch runs while the statement branch's first features and weights are on their way, in
// LDS that this branch's tiles take over; the head's weights are requested when the last statement tile has left their registers.
// Bound: latency, a launch and the chain of three stages with few tiles each (of three launches, each waited for the one before,
// loaded its weights and drained).  A call, three launches -> one: 100 candidates 29.6 -> 23.3 us, 2,048 30.5 -> 24.2, 8,192
// 36.7 -> 27.7, 16,384 51.4 -> 42.9.  (With the dataflow branch before the statement counts are numbered 8,192 took 29.7.)

constexpr int kSmallMost = kTM;   // candidates of a workgroup

static_assert(sizeof(FlowLds<kSmallMost>) <= kArena * sizeof(__bf16), "the dataflow branch's LDS is the statement branch's arena");

__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(1, 1)))
pacm_small_kernel(const float* __restrict__ feat, const int32_t* __restrict__ n_stmt, const float* __restrict__ flow, const int32_t* __restrict__ n_blk,
                  int32_t n_d, pruner_pacm w, float* __restrict__ y)
{
    __shared__ __attribute__((aligned(16))) __bf16 arena[kArena];
    __shared__ __attribute__((aligned(16))) float cst[2][kH];
    __shared__ uint16_t before[kSmallMost + 64 + 2];
    __shared__ int32_t row_src[kTM];
    __shared__ uint32_t scan_tot[4];
    __shared__ __attribute__((aligned(16))) __bf16 U[(kTM + 1) * kUs];   // the concatenated pooled vectors
    __shared__ __attribute__((aligned(16))) float bh_lds[kH];
    __shared__ __attribute__((aligned(16))) uint16_t wo_lds[kH];
    __shared__ float red[4][kTM];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int half = lane >> 5, l32 = lane & 31;
    const Share share(n_d, kGroupMinLog, (int)blockIdx.x, (int)gridDim.x);
    // the wavefront's candidates in the dataflow branch
    const int per = (share.n_local + kFlowWaves - 1) / kFlowWaves, from = wave * per < share.n_local ? wave * per : share.n_local;
    const int mine = from + per < share.n_local ? per : share.n_local - from;
    const int blk_count = lane < mine ? n_blk[share.global_of(from + lane)] : 0;
    const float bh_mine = w.bh[threadIdx.x];
    const uint16_t wo_mine = w.wo[threadIdx.x];
    FlowWeights flow_weights;
    flow_weights.load(w.We, w.be, w.Wq, w.Wk, w.Wv, w.Wo, wave, l32, half);
    stmt_branch<true>(StmtLds{arena, cst, before, row_src, scan_tot}, share, feat, n_stmt, w.W1, w.b1, w.W2, w.b2, PooledToLds{U}, [&]() {
        bh_lds[threadIdx.x] = bh_mine;
        wo_lds[threadIdx.x] = wo_mine;
        flow_branch(reinterpret_cast<FlowLds<kSmallMost>&>(arena), mine, [&](int l) { return share.global_of(from + l); },
                    [&](int l) { return reinterpret_cast<uint16_t*>(U) + (from + l) * kUs + kH; }, flow, n_blk, blk_count, flow_weights);
    });
    bf16x8 whr[2][kU / 16];
    load_slices<kU / 16, kU / 16, u32x4>(whr, w.Wh, kU, wave, l32, half);
    float wor[2][16];   // this lane's output weights, in accumulator order
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
        for (int i = 0; i < 16; ++i) wor[nt][i] = __uint_as_float((uint32_t)wo_lds[64 * wave + 32 * nt + 8 * (i / 4) + 4 * half + (i % 4)] << 16);
    __syncthreads();   // the pooled vectors are complete
    for (int row0 = 0; row0 < share.n_local; row0 += 32) {
        floatx16 acc[2];
        bias_init(acc, bh_lds, wave, half);
        layer<kU / 16>(acc, whr, U + row0 * kUs, kUs, l32, half, [](int) {});
        float part = 0.f;
#pragma unroll
        for (int pair = 0; pair < 16; ++pair) {
            const int nt = pair >> 3, p = pair & 7;
            const uint32_t pr = relu_bf16x2(acc[nt][2 * p], acc[nt][2 * p + 1]);
            part = __builtin_fmaf(__uint_as_float(pr << 16), wor[nt][2 * p], part);
            part = __builtin_fmaf(__uint_as_float(pr & 0xFFFF0000u), wor[nt][2 * p + 1], part);
        }
        part += __shfl_xor(part, 32, 64);
        if (half == 0) red[wave][row0 + l32] = part;
    }
    __syncthreads();
    if ((int)threadIdx.x < share.n_local)
        y[share.global_of((int)threadIdx.x)] = (((red[0][threadIdx.x] + red[1][threadIdx.x]) + red[2][threadIdx.x]) + red[3][threadIdx.x]) + w.bo;
}

}  // namespace

// (binary32 pooled vectors' room, of which the bfloat16 ones take half: the size that callers know)
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
    // One launch as long as a workgroup's pooled vectors are one tile of the head (16,384 candidates on this part, 51.4 -> 42.9 us; LDS
    // has no room for a second tile beside the statement branch's).
    if (n_d <= (int64_t)kSmallMost * pacm_cus) {
        const int64_t grid = (n_d + kGroupMin - 1) / kGroupMin < pacm_cus ? (n_d + kGroupMin - 1) / kGroupMin : pacm_cus;
        hipLaunchKernelGGL(pacm_small_kernel, dim3((unsigned)grid), dim3(kThreads), 0, st, feat, n_stmt, flow, n_blk, n, *w, y);
        PRUNER_LAUNCH_CHECK();
        return PRUNER_OK;
    }
    // statement branch: one launch per kLocalCap x (compute units) candidates, groups as in pruner_verify_score
    const int64_t per_launch = (int64_t)kLocalCap * pacm_cus;
    for (int64_t c0 = 0; c0 < n_d; c0 += per_launch) {
        const int64_t m = n_d - c0 < per_launch ? n_d - c0 : per_launch;
        const int64_t grid = (m + kGroupMin - 1) / kGroupMin < pacm_cus ? (m + kGroupMin - 1) / kGroupMin : pacm_cus;
        int group_log = kGroupMinLog;
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
