// Host-side launch interface between the C-ABI layer (api.hip) and the kernel files.
#pragma once
#include <hip/hip_ext.h>

#include "common.hpp"

namespace fastocr {

// Kernel ids mirror fastocr_kernel in fastocr.h (used by the per-kernel timers).
enum KernelId {
    K_SCORE_LOGITS = 0, K_SCORE_FINALIZE = 1, K_TOPK = 2, K_SPARSE_ATTN = 3, K_DENSE_ATTN = 4,
    K_ATTN_COMBINE = 5, K_FOCAL_FUSED = 6, K_PARKED_FINISH = 7, K_COUNT = 8
};

// Per-kernel timing (api.hip): when a timer is enabled for `kernel`, the next launch gets a pair of
// events that the runtime stamps at the kernel's own start and end (hipExtLaunchKernelGGL);
// otherwise both are null and the launch is an ordinary one.
struct TimerEvents { hipEvent_t start, stop; };
TimerEvents timer_events(int kernel);

#define FASTOCR_LAUNCH(KID, KERNEL, GRID, BLOCK, SHMEM, STREAM, ...)                                   \
    do {                                                                                               \
        const ::fastocr::TimerEvents te_ = ::fastocr::timer_events(KID);                               \
        hipExtLaunchKernelGGL((KERNEL), (GRID), (BLOCK), (SHMEM), (STREAM), te_.start, te_.stop, 0,    \
                              __VA_ARGS__);                                                            \
    } while (0)

enum { DT_F32 = 0, DT_BF16 = 1 };

struct Shape {
    KvDev kv;
    BatchDev bv;
    int batch;
    int n_q_heads;
    int dtype;
    bool paged;
    bool vec16;     // every cache row starts 16-byte aligned and head_dim covers whole 16-byte pieces
    bool fast;      // the MFMA kernels cover this shape: bf16, head_dim 128 or 64, group size <= 16,
                    // 16-byte aligned rows (decided once from the views by the C-ABI layer)
    bool fast32;    // the fp64 matrix-core kernels of attn_f32.hip cover it: fp32, head_dim 128 or 64, group size <= 16, vec16
};

inline bool mfma_path(const Shape &s) { return s.fast; }
inline bool f32_mfma_path(const Shape &s) { return s.fast32; }

// ---- host-side state shared by the launchers (api.hip) --------------------------------------
// Launch-shape overrides (fastocr_set_tuning); atomics, so that callers on several threads may
// read them while another thread sets one.
int tune_attn_waves();                 // 4 or 8
long long tune_spin_ticks();           // bounded wait of the single-launch forms, in 100 MHz wall-clock ticks
// Compute units the launch shapes are planned for: the current device's, or 256 (MI355X) when no
// device can be asked.
int plan_cu_count();

// Exchange slots of the single-launch forms.  Workgroups of such a launch hand each other data
// through static device memory, one slot per call in flight.  Two calls may share a slot only if
// the second cannot start before the first has ended, i.e. if they are enqueued on the same
// stream; so a slot belongs to a stream: the first k*EagerSlots streams of a device that ask for
// one keep it for the life of the process.  A call that is being captured into a HIP graph gets a
// slot of a separate pool that belongs to (capture, stream) and is never handed out again -- the
// graph may be replayed on any stream next to eager calls.  Returns the slot, or -1 when none is
// left (or the stream's capture state cannot be read): the caller then takes the form built from
// separate kernels, which shares nothing.
enum ExchangeKind { EX_SCORE = 0, EX_FUSED = 1, EX_MERGE = 2, EX_KINDS = 3 };
constexpr int kResSlots = 64;          // slots of each register-resident kernel (scoring, fused focal layer), 128 KB of static memory each
constexpr int kResEagerSlots = 16;     //   of which for streams; the rest for graph captures
constexpr int kMergeSlots = 16;        // slots of pruned attention's in-launch merge, 3.2 MB of static memory each
constexpr int kMergeEagerSlots = 4;
// *gave_up_flag: a device-visible word in pinned host memory that a wave sets when it gives up
// waiting inside a single-launch form (null if it could not be allocated yet: the first call on a
// device happened inside a capture); once it is set the library's own choice (tuning mode 1) is
// the separate-kernel forms for the rest of the process ("exchange_fallback" 0 re-arms it).
int exchange_slot(int kind, hipStream_t stream, uint32_t **gave_up_flag);
bool exchange_trusted();               // false once a wave has given up (or "exchange_fallback" 1)

// Image-mass partials to be summed per sequence (out == nullptr: none): n_part per sequence, or with seq_meta one
// per workgroup of the one-pass focal kernel.
struct MassArgs {
    const float *part;
    float *out;                 // [B]
    int n_part;
};

// The top-k inside a launch that finishes scores (sel_idx == nullptr: none): the arguments of fastocr_topk_fixation.
struct SelectArgs {
    double tau;
    const int32_t *prev_idx, *prev_cnt;
    int32_t *sel_idx, *sel_cnt;
    int64_t kmax;
};

// ---- attention (attn.hip) ---------------------------------------------------------------
// Workspace: part_o fp32 [B][Hq][nsplit][d] followed by part_ml fp32 [B][Hq][nsplit][2].
int attn_tile_tokens(const Shape &s);
size_t attn_workspace_bytes(const Shape &s, size_t rows);             // rows = B * Hq * nsplit
// With 2 .. 4 ranges per stream on the MFMA path the stream's last range can merge the others'
// partials inside the launch (through static device memory) when the shape fits
// (attn_merges_in_kernel) and an exchange slot is given; otherwise partials go to the workspace
// and a merge kernel follows.
bool attn_merges_in_kernel(const Shape &s, int nsplit);
// merge_slot of a call whose ranges would merge inside the launch if a slot were left: partials and the merge kernel, with the
// merging kernel's tiles and roundings, so that the outputs' bits do not depend on how many streams are in use.
constexpr int kNoMergeSlot = -2;
// merge_slot: exchange slot for the in-launch merge (EX_MERGE), or -1 = partials + merge kernel.
hipError_t launch_attn(const Shape &s, const void *q, float scale, const int32_t *sel_idx,
                       const int32_t *sel_cnt, int64_t kmax, void *out, float *lse, void *ws,
                       int nsplit, int merge_slot, uint32_t *gave_up_flag, hipStream_t stream);
// Pruned attention of n <= kLayerSet layers in one launch: caches shaped like s.kv at their own places, one kept set, s.fast.  nsplit: 1, or a range
// count that merges inside the launch (attn_merges_in_kernel of a shape with n times the sequences, merge_slot then >= 0).
// kLayerSet: the layers' pointers are kernel arguments, 40 bytes each (us with 4 / 8 / 16 / 32 layers a launch, one by one; 26 layers of 28/4 heads, batch 8, 420 rows
// 66.3 / 46.9 / 39.8 / 34.9, 218; batch 1 61.3 / 35.6 / 19.2 / 13.8, 208; 33 layers of 16/2, batch 12, 840 rows 112 / 80.4 / 71.9 / 63.4, 313; 26 of
// 64/8, batch 16, 840 rows 247 / 236 / 229 / 229, 372).
constexpr int kLayerSet = 32;
struct LayerPtrs { const void *k, *v, *q; void *out; const int32_t *block_table; };
hipError_t launch_attn_layers(const Shape &s, int n, const LayerPtrs *at, float scale, const int32_t *sel_idx, const int32_t *sel_cnt,
                              int64_t kmax, int nsplit, int merge_slot, uint32_t *flag, hipStream_t stream);
// Dense attention whose logits of the image tokens stay behind in `logits` (fp32, log2 domain, [sequence][query head][pitch]);
// always partials.  part_o == nullptr: logits and statistics alone.  part_zi: the image tokens' part of every range's sum-exp,
// [rows], or null.  zero: [batch] words the launch clears, or null.  Shapes with parks_by_head.
hipError_t launch_attn_parked(int kid, const Shape &s, const void *q, float scale, float *part_o, float *part_ml, float *part_zi,
                              int nsplit, float *logits, int64_t pitch, uint32_t *zero, hipStream_t stream);
// merge of nsplit partials per (sequence, head) in the layout above into the final output.
// With seq_meta (device int32 [B][2]: first workgroup, workgroup count) the partials are instead
// those of the fused focal kernel, [workgroup][wpk][Hq][d] / [..][2], wpk per workgroup.
// mass: the launch also sums the image-mass partials of every sequence.
hipError_t launch_attn_combine(const Shape &s, const float *part_o, const float *part_ml, int nsplit,
                               void *out, float *lse, hipStream_t stream, const int32_t *seq_meta = nullptr,
                               int wpk = 1, MassArgs mass = MassArgs{nullptr, nullptr, 0});

// ---- fp32 caches on the fp64 matrix cores (attn_f32.hip; shapes with s.fast32) --------------
// sel_idx: pruned attention.  part_o == nullptr: no attention output.  logits: the logits are parked there (with
// row pitch `pitch`) for the score kernels.  nsplit == 1 without logits: the kernel writes the final output itself.
hipError_t launch_attn_f32(int kid, const Shape &s, const void *q, float scale, const int32_t *sel_idx, const int32_t *sel_cnt,
                           int64_t kmax, float *part_o, float *part_ml, int nsplit, void *out, float *lse, float *logits,
                           int64_t pitch, hipStream_t stream);

// ---- focal scoring (score.hip) ----------------------------------------------------------
// Workspace: logits fp32 [B][Hq][pitch], part_ml fp32 [B][Hq][nsplit][2], image sums or mass partials.
size_t score_workspace_bytes(const Shape &s, size_t rows);            // rows = B * Hq * nsplit
hipError_t launch_score(const Shape &s, const void *q, float scale, float *scores, float *lse,
                        float *img_mass, void *ws, int nsplit, hipStream_t stream, const SelectArgs *select = nullptr);

// Where a row's parked logits are read for the tokens p .. p + 3 (p a multiple of 4): past the pitch its last four, which nobody uses.
// A batch of empty sequences alone has a pitch of 0: its reads meet the statistics, which follow the logits and are at least as large.
__host__ __device__ inline int parked_token(int p, int64_t pitch) { return max(0, min(p, (int)pitch - 4)); }

struct CombineArgs;
bool parks_by_head(const Shape &s);    // the matrix-core kernels of attn.hip park this shape's logits
// A focal layer of a bf16 cache as two launches that wait for nothing (parks_by_head).  nsplit: that of dense attention.
// select: the second launch does the top-k too (image spans of up to 16384 tokens, as in launch_score); defer (without
// select): see launch_focal_fused; the image mass is not handed on.
size_t focal_parked_workspace_bytes(const Shape &s, size_t rows);     // rows = B * Hq * nsplit
hipError_t launch_focal_parked(const Shape &s, const void *q, float scale, void *out, float *scores, float *lse, float *img_mass,
                               void *ws, int nsplit, hipStream_t stream, const SelectArgs *select = nullptr, CombineArgs *defer = nullptr);

// A focal layer of an fp32 cache in one pass (s.fast32): attention partials and parked logits from one read of K
// and V, then the scores.  nsplit: that of dense attention.  defer: see launch_focal_fused.
size_t focal_f32_workspace_bytes(const Shape &s, size_t rows);        // rows = B * Hq * nsplit
hipError_t launch_focal_f32(const Shape &s, const void *q, float scale, void *out, float *scores, float *lse, float *img_mass,
                            void *ws, int nsplit, hipStream_t stream, CombineArgs *defer = nullptr);

// ---- focal scoring with register-resident logits (score_resident.hip) ---------------------
// The plan gives the grid (nranges * batch workgroups, at most one per compute unit) and the
// range length used when all sequences are equally long; ragged batches are split on the device.
// Workspace, W = nranges * batch: image-mass partials fp32 [W], per sequence its first workgroup
// and range count int32 [B][2] (the ranges' softmax statistics travel through static device memory).
struct ResidentPlan { int nranges, range_tokens, wpk; };
// whether the fused select covers the shape (image spans of up to 16384 tokens)
bool resident_select_fits(const Shape &s);
bool resident_plan(const Shape &s, int num_cu, ResidentPlan *plan);
// The most workgroups a plan of this cache for at most these sequences has, in number and length (0: never a plan).
int resident_max_workgroups(const Shape &s, int num_cu);
size_t resident_workspace_bytes(const Shape &s, const ResidentPlan &p);
hipError_t launch_score_resident(const Shape &s, const ResidentPlan &p, int sync_slot, uint32_t *gave_up_flag, const void *q, float scale,
                                 float *scores, float *lse, float *img_mass, void *ws, hipStream_t stream,
                                 const SelectArgs *select = nullptr);

// ---- focal layer in one pass: dense attention output + scores (focal_fused.hip) -----------
// Uses the same plan as the register-resident scoring kernel.
size_t focal_fused_workspace_bytes(const Shape &s, int num_cu);
// A merge of attention partials handed on to the launch that follows (see launch_topk).
struct CombineArgs {
    const float *part_o, *part_ml;
    int nsplit, d, n_q_heads, wpk;
    const int32_t *seq_meta;    // null: nsplit partials per (sequence, head), see launch_attn
    void *out;                  // [B, Hq, d]: bf16, or fp32 with out_f32
    bool out_f32;
    MassArgs mass;              // the image-mass partials to sum on the way (mass.out null: none)
};
// defer != nullptr: the merge of the output's partials is not launched; *defer describes it and the
// caller passes it to launch_topk, whose launch then does both (the top-k and that merge depend on
// this kernel only, not on each other), and sums the image mass.
hipError_t launch_focal_fused(const Shape &s, const ResidentPlan &p, int sync_slot, uint32_t *gave_up_flag, const void *q, float scale,
                              void *out, float *scores, float *lse, float *img_mass, void *ws, hipStream_t stream,
                              const SelectArgs *select = nullptr, CombineArgs *defer = nullptr);

// ---- how often a workgroup gave up waiting for another one of its launch (each file's own count;
// the copies synchronise with the device) ----------------------------------------------------
hipError_t score_resident_timeouts(uint32_t *n);
hipError_t focal_fused_timeouts(uint32_t *n);
hipError_t attn_merge_timeouts(uint32_t *n);

// ---- top-k (topk.hip) -------------------------------------------------------------------
size_t topk_workspace_bytes(int batch, int max_vis_len);
// combine != nullptr (only when topk_takes_combine says so): the launch gets one more workgroup per
// (sequence, query head), which merges that head's attention partials.
hipError_t launch_topk(const float *scores, const BatchDev &bv, int batch, double tau,
                       const int32_t *prev_idx, const int32_t *prev_cnt, int32_t *sel_idx,
                       int32_t *sel_cnt, int64_t kmax, void *ws, hipStream_t stream,
                       const CombineArgs *combine = nullptr);
bool topk_takes_combine(int max_vis_len, int head_dim);

// ---- streaming probe (probe.hip) ----------------------------------------------------------
hipError_t launch_stream_probe(const void *src, void *dst, size_t bytes, void *sink, hipStream_t stream);

}  // namespace fastocr
