// Internal helpers shared by the entry points of the HIP library (not part of the C boundary).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <vector>

#include "pruner.h"

namespace pruner {

constexpr int kWave = 64;  // gfx950 wavefront

inline bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }
inline size_t round_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Inclusive prefix sum over the 64 lanes of a wavefront (every lane active).  Data-parallel-primitive adds: shifts by
// 1, 2, 4 and 8 lanes inside each row of 16 lanes, then lane 15 of rows 0 and 2 into rows 1 and 3, then lane 31 into
// rows 2 and 3; a lane without a source adds 0.  Six full-rate vector instructions where shuffles through LDS
// hardware take six round trips.
__device__ __forceinline__ uint32_t wave_inclusive_sum(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);   // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);   // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);   // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);   // row_shr:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1, 3
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2, 3
    return v;
}

// Inclusive running maximum over the active lanes of a wavefront, by the same moves: the last active lane ends up
// with the maximum of all active lanes when these are lanes 0..m (a lane without a source, or whose source is switched
// off, keeps its own value).  In two parts: inside each row of 16 lanes, then across the rows.
template <int CTRL, int ROWS> __device__ __forceinline__ uint32_t max_with(uint32_t v)
{
    const uint32_t y = (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, ROWS, 0xf, false);
    return v > y ? v : y;
}
__device__ __forceinline__ uint32_t row_inclusive_max(uint32_t v)
{
    return max_with<0x118, 0xf>(max_with<0x114, 0xf>(max_with<0x112, 0xf>(max_with<0x111, 0xf>(v))));
}
__device__ __forceinline__ uint32_t rows_inclusive_max(uint32_t v) { return max_with<0x143, 0xc>(max_with<0x142, 0xa>(v)); }
__device__ __forceinline__ uint32_t wave_inclusive_max(uint32_t v) { return rows_inclusive_max(row_inclusive_max(v)); }

// After a launch: PRUNER_EHIP if the runtime reports an error.  hipGetLastError returns (and clears) the last error
// of the calling thread, so an error left by an earlier, unrelated runtime call is reported here as well; launches that
// came before in the same call stay enqueued.
#define PRUNER_LAUNCH_CHECK()                      \
    do {                                           \
        if (hipGetLastError() != hipSuccess) return PRUNER_EHIP; \
    } while (0)

// Facts about the current device that entry points look up once per device: the number of its compute units, and
// whether a kernel's attribute has been set on it (function attributes belong to the device the call was made on).
// Devices are told apart by their ordinal; the tables hold kMaxDevices of them, later ordinals are looked up every time.
constexpr int kMaxDevices = 64;
int current_device(int* compute_units);   // the ordinal (and the count), or -1 if the runtime reports an error
struct PerDeviceFlag {
    bool set[kMaxDevices] = {};
    bool get(int dev) const { return dev >= 0 && dev < kMaxDevices && set[dev]; }
    void mark(int dev) { if (dev >= 0 && dev < kMaxDevices) set[dev] = true; }
};

// Stream-ordered copy of a small host table into device memory without staging buffers: the bytes travel as
// kernel arguments (copied by the runtime at launch), so the host copy may be freed as soon as the call returns
// and the launch can be captured into a graph.
constexpr int kPutBytes = 4032;   // with the kernel's other arguments below the 4 KB that a launch carries
struct PutPayload {
    uint4 q[kPutBytes / 16];
};
// Optionally the same launch clears zero_bytes of device scratch at zero_device.
int put_table(void* dst_device, const void* src_host, size_t bytes, hipStream_t stream, void* zero_device = nullptr,
              size_t zero_bytes = 0);

// A table upload that has been prepared but not launched: a later upload into the same workspace takes it along
// (one launch instead of two).
struct Upload {
    std::vector<char> bytes;
    void* dst = nullptr;
    void* zero = nullptr;
    size_t zero_bytes = 0;
};

// Selection in two steps, so that a caller inside the library can produce the first-digit histograms itself
// between them (the draft kernel does, while the scores are still in registers).
struct TopkCtx {
    bool digits;           // the route counts first digits (lists and spans)
    bool tiny, pick, levels, blocks_route, lists;   // the route; none of them: spans
    int32_t n_sg, k;
    int64_t n, longest, span;
    int share;             // workgroups that rank a segment's words
    bool sort;             // ... or sort them, if they are many
    int32_t blocks;        // workgroups of a sweep launch
    int copies;            // copies of the first digit's histogram
    void *d_segs, *d_state, *d_stage, *d_parts;
    uint32_t* d_hist;      // [copies][n_sg][2048] first digit, then one copy each for the second and third
    uint32_t* d_max256;    // largest key of every 256 neighbouring entries (block_max_slot), or null: the route does without
    uint32_t *d_max64, *d_max16;   // ... of every 64 (block64_slot) and 16 (block16_slot), or null
    char inline_segs[4096];  // tiny, pick and levels: the segment table when it travels as a kernel argument
    bool inline_ok;
};
// What the selection would have whoever holds the scores in registers leave behind (null pointers: nothing of the kind).
struct ScoreNotes {
    uint32_t* first_digit = nullptr;   // every score's first digit added to one of `copies` histograms
    int copies = 1;
    uint32_t *max256 = nullptr, *max64 = nullptr, *max16 = nullptr;   // (with the first digits: the former alone; else the latter and the others as well)
};
inline ScoreNotes notes_for(const TopkCtx& ctx) { return ScoreNotes{ctx.digits ? ctx.d_hist : nullptr, ctx.copies, ctx.d_max256, ctx.d_max64, ctx.d_max16}; }
// validates, uploads the segment table, clears the histograms (of the routes that count digits)
// (defer: do not launch the upload, describe it there instead; copies: the scores are expected to hold ties by the thousand)
int topk_prepare(const int64_t* seg_off, int32_t n_sg, int32_t k, void* workspace, size_t workspace_bytes, hipStream_t stream, TopkCtx* ctx,
                 Upload* defer, bool with_block_max, bool copies);
// the remaining launches; noted: what notes_for(ctx) asks for is in place
int topk_finish(const TopkCtx& ctx, const float* score, const int64_t* seg_off, int32_t* idx_out, float* val_out, bool noted,
                hipStream_t stream);

// Everything pruner_draft_score refuses, without enqueuing anything.
int draft_check(const pruner_subgraph* sg, int32_t n_sg, const int64_t* seg_off, const uint16_t* tiles, int64_t tiles_pitch, int32_t flags,
                const float* score, const int64_t* symbols, const void* workspace, size_t workspace_bytes);
struct MutArgs;   // lse_child.h

// The draft launches of a call: planned once (everything pruner_draft_score refuses is refused here), their tables, where they are
// too large for the launches to bring along, uploaded to the workspace's begin, then run, as often as the population's shape stays the same.
struct DraftPlan {
    struct Launch {
        int cls;
        int32_t first_seg, n_seg;
        int64_t blocks, candidates, bytes;   // workgroups; candidates and their algorithmic bytes
        const void *fn, *fn_read;            // the kernel; the same without making its candidates
    };
    std::vector<Launch> launches;
    std::vector<char> image;   // the tables
    size_t descs_at = 0;
    bool in_launch = false;    // they travel with the launches themselves and are not uploaded (draft_upload decides)
    int64_t n = 0, tiles_pitch = 0;
    int32_t n_sg = 0, flags = 0, n_classes = 0;   // (loop-nest classes)
    bool exact = false;    // one rounded operation per step of Eq. 1
    bool makes = false;    // the kernels can make their candidates (the explorer loop's mutation) instead of reading them
};
// notes: what the selection would have the kernels leave behind; mut: the kernels
// are to make their candidates from the second run on (plan->makes says whether they can): the children of S_spec as they are drawn, the same
// where all their scores are looked up, or all that S_spec can have.
enum class Makes { kNothing, kChildren, kLookedUp, kVariants };
int draft_plan(const pruner_subgraph* sg, int32_t n_sg, const int64_t* seg_off, const uint16_t* tiles, int64_t tiles_pitch, int32_t flags,
               const float* score, const int64_t* symbols, const void* workspace, size_t workspace_bytes, const ScoreNotes& notes, Makes mut, DraftPlan* plan);
// (also: an upload prepared by someone else whose destination lies in the same allocation shortly after the plan's own tables
// and behind which nothing else lies that must stay.  An upload that begins right behind the tables (place_behind) shares
// their launch.
int draft_upload(DraftPlan& plan, void* workspace, hipStream_t stream, const Upload* also);
bool fits_launch(const DraftPlan& plan);   // the tables are small enough to travel with the launches
// Moves the pending table to the first free place behind the plan's tables in the same workspace (it was prepared for a later
// one, so it fits); returns where it will lie.
void* place_behind(const DraftPlan& plan, void* workspace, Upload* also);
// Draft scores, and what `notes` asks for (as the plan was made for).  mut (needs plan.makes): the kernels make the children of
// S_spec and score them (`tiles` stays as it is), or score all children that S_spec can have, or look the children's scores up there.
int draft_run(const DraftPlan& plan, const void* workspace, const uint16_t* tiles, float* score, int64_t* symbols, hipStream_t stream,
              const ScoreNotes& notes, const MutArgs* mut);
// workspace needs of the entry points (each defined next to its kernels)
size_t draft_workspace_bytes(int32_t n_sg);
size_t topk_workspace_bytes(int64_t n, int32_t n_sg, int32_t k, bool parts);   // parts: with room for the lists of the blocks route, which a call can do without
size_t verify_workspace_bytes(int64_t n_d);
size_t prior_filter_workspace_bytes(int64_t n, int32_t n_sg, int32_t k, bool parts);
size_t lse_workspace_bytes(int64_t n, int32_t n_sg, int32_t k, int32_t rows);
size_t pacm_workspace_bytes(int64_t n_d);

}  // namespace pruner
