// C ABI of the FastOCR decode hot path: host-side validation, workspace sizing, launch-shape
// choice and per-kernel event timers.  Every check happens before the first HIP call, so the
// error paths can be exercised without a GPU.
#include <math.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <mutex>
#include <vector>

#include "apart.hpp"
#include "fastocr.h"
#include "kernels.hpp"

namespace fastocr {

// ---- launch-shape overrides (fastocr_set_tuning) --------------------------------------------
// Plain values read on every call and written rarely, possibly from another thread: atomics.
static std::atomic<int> g_tune_score_resident{1};
static std::atomic<int> g_tune_focal_fused{1};
static std::atomic<int> g_tune_attn_waves{4};
static std::atomic<int> g_tune_attn_merge{1};          // pruned attention: ranges of a stream merged inside the launch (0 never, 1 yes)
static std::atomic<int> g_tune_barrier_spin_us{250000};      // bounded wait of the single-launch forms
static std::atomic<int> g_tune_splits[4];              // indexed by fastocr_op; 0 = automatic
static std::atomic<int> g_tune_timer_every{1};         // per-kernel timers: which launches record events (every n-th)
static std::atomic<int> g_exchange_distrusted{0};      // "exchange_fallback" 1
static std::atomic<int> g_tune_graph_replay{0};        // 1: the caller replays its calls from a HIP graph, where a launch follows the one before within half a microsecond
static std::atomic<int> g_tune_select_fused{0};        // top-k inside the scoring / focal-layer launch (0 never, 1 when it fits): measured slower, off by default

int tune_attn_waves() { return g_tune_attn_waves.load(std::memory_order_relaxed); }
long long tune_spin_ticks() { return 100ll * g_tune_barrier_spin_us.load(std::memory_order_relaxed); }   // the wall clock runs at 100 MHz

// Everything below that is more than one word (timers, slot registry, per-device tables) is
// guarded by one mutex; it is held for a few table look-ups per call.
static std::mutex g_mu;

// ---- per-kernel timers ------------------------------------------------------------------
struct KernelTimer {
    int capacity = 0;
    int count = 0;
    unsigned seen = 0;      // launches of the kernel since the timer was enabled
    hipEvent_t *start = nullptr;
    hipEvent_t *stop = nullptr;
};
static KernelTimer g_timers[K_COUNT];

TimerEvents timer_events(int kernel)
{
    std::lock_guard<std::mutex> lock(g_mu);
    KernelTimer &t = g_timers[kernel];
    if (t.count >= t.capacity) return TimerEvents{nullptr, nullptr};
    // an event pair costs the stream a few microseconds: only every timer_every-th launch carries one
    if (t.seen++ % (unsigned)g_tune_timer_every.load(std::memory_order_relaxed) != 0u) return TimerEvents{nullptr, nullptr};
    const int i = t.count++;
    return TimerEvents{t.start[i], t.stop[i]};
}

// ---- the device the call runs on ----------------------------------------------------------------
constexpr int kMaxDevices = 64;

static int current_device()
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) { (void)hipGetLastError(); return -1; }
    return dev >= 0 && dev < kMaxDevices ? dev : -1;
}

int plan_cu_count()
{
    static int cached[kMaxDevices] = {0};          // 0 = not asked yet; guarded by g_mu
    const int dev = current_device();
    if (dev < 0) return 256;
    std::lock_guard<std::mutex> lock(g_mu);
    if (cached[dev] == 0) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) { (void)hipGetLastError(); n = 0; }
        cached[dev] = n > 0 ? n : 256;
    }
    return cached[dev];
}

// ---- exchange slots (see kernels.hpp) --------------------------------------------------------------
struct SlotOwner { hipStream_t stream; unsigned long long capture; bool free; };
struct SlotTable { std::vector<SlotOwner> eager, graph; };
static SlotTable g_slots[EX_KINDS][kMaxDevices];

static uint32_t *g_gave_up[kMaxDevices];       // pinned host memory, one word per device, never freed

int exchange_slot(int kind, hipStream_t stream, uint32_t **gave_up_flag)
{
    *gave_up_flag = nullptr;
    const int total = kind == EX_MERGE ? kMergeSlots : kResSlots;
    const int n_eager = kind == EX_MERGE ? kMergeEagerSlots : kResEagerSlots;
    const int dev = current_device();
    if (dev < 0) return -1;
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    unsigned long long cap = 0;
    if (hipStreamGetCaptureInfo(stream, &st, &cap) != hipSuccess) {
        // e.g. the legacy default stream while another stream of the device is capturing
        (void)hipGetLastError();
        return -1;
    }
    if (st == hipStreamCaptureStatusInvalidated) return -1;
    const bool capturing = st == hipStreamCaptureStatusActive;
    std::lock_guard<std::mutex> lock(g_mu);
    if (!g_gave_up[dev] && !capturing) {
        // one word of pinned host memory per device, allocated on the first eager call that reaches
        // this point (an allocation is not a capturable call) and kept until the process ends
        void *p = nullptr;
        if (hipHostMalloc(&p, 64, hipHostMallocMapped | hipHostMallocCoherent) == hipSuccess && p) {
            memset(p, 0, 64);
            g_gave_up[dev] = static_cast<uint32_t *>(p);
        } else {
            (void)hipGetLastError();
        }
    }
    *gave_up_flag = g_gave_up[dev];
    SlotTable &t = g_slots[kind][dev];
    std::vector<SlotOwner> &pool = capturing ? t.graph : t.eager;
    const int cap_n = capturing ? total - n_eager : n_eager;
    const int first = capturing ? n_eager : 0;
    for (size_t i = 0; i < pool.size(); ++i)
        if (!pool[i].free && pool[i].stream == stream && (!capturing || pool[i].capture == cap)) return first + (int)i;
    for (size_t i = 0; i < pool.size(); ++i)
        if (pool[i].free) {                      // released by fastocr_stream_release
            pool[i] = SlotOwner{stream, capturing ? cap : 0ull, false};
            return first + (int)i;
        }
    if ((int)pool.size() >= cap_n) return -1;
    pool.push_back(SlotOwner{stream, capturing ? cap : 0ull, false});
    return first + (int)pool.size() - 1;
}

bool exchange_trusted()
{
    if (g_exchange_distrusted.load(std::memory_order_relaxed)) return false;
    const int dev = current_device();
    if (dev < 0) return true;
    std::lock_guard<std::mutex> lock(g_mu);
    const uint32_t *f = g_gave_up[dev];
    return !f || __atomic_load_n(f, __ATOMIC_RELAXED) == 0u;
}

// ---- workspace in static device memory, for fastocr_dense_decode_attn_static -------------------------
// The array's name is a host-side handle, not a device address: what kernels and copies get is the
// address hipGetSymbolAddress returns for the device that is current, asked for once per device
// (every GPU holds its own copy of the array at its own address).
static __device__ __align__(256) unsigned char scratch[FASTOCR_STATIC_SCRATCH_BYTES];
static void *g_scratch_ptr[kMaxDevices];       // guarded by g_mu

static void *static_scratch_ptr()
{
    const int dev = current_device();
    if (dev < 0) return nullptr;
    std::lock_guard<std::mutex> lock(g_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) { (void)hipGetLastError(); return nullptr; }
        g_scratch_ptr[dev] = p;
    }
    return g_scratch_ptr[dev];
}

// ---- shapes -----------------------------------------------------------------------------
static int check_views(const fastocr_kv_view *kv, const fastocr_batch_view *bv, int n_q_heads)
{
    if (!kv || !bv) return FASTOCR_EINVAL;
    if (!kv->k || !kv->v) return FASTOCR_EINVAL;
    if (kv->dtype != FASTOCR_F32 && kv->dtype != FASTOCR_BF16) return FASTOCR_EUNSUPPORTED;
    if (kv->n_kv_heads < 1 || kv->head_dim < 1) return FASTOCR_EINVAL;
    if (n_q_heads < 1 || n_q_heads % kv->n_kv_heads != 0) return FASTOCR_EINVAL;
    if (kv->head_dim > 256 || n_q_heads > 256) return FASTOCR_EUNSUPPORTED;
    if (kv->stride_token < kv->head_dim || kv->stride_head < 0 || kv->stride_seq < 0) return FASTOCR_EINVAL;
    if (bv->batch < 0 || bv->max_seq_len < 0 || bv->max_vis_len < 0) return FASTOCR_EINVAL;
    if (bv->max_vis_len > bv->max_seq_len) return FASTOCR_EINVAL;
    if (bv->batch > 65535) return FASTOCR_EUNSUPPORTED;
    if (bv->batch > 0 && (!bv->seq_len || !bv->vis_start || !bv->vis_len)) return FASTOCR_EINVAL;
    if (kv->page_tokens < 0) return FASTOCR_EINVAL;
    if (kv->page_tokens > 0) {
        if (!kv->block_table || kv->stride_page < 1) return FASTOCR_EINVAL;
        const int64_t need = ((int64_t)bv->max_seq_len + kv->page_tokens - 1) / kv->page_tokens;
        if (kv->max_pages_per_seq < need || kv->max_pages_per_seq < 1) return FASTOCR_EINVAL;
    }
    return FASTOCR_OK;
}

static Shape make_shape(const fastocr_kv_view *kv, const fastocr_batch_view *bv, int n_q_heads)
{
    Shape s;
    s.kv.k = kv->k;
    s.kv.v = kv->v;
    s.kv.stride_token = kv->stride_token;
    s.kv.stride_head = kv->stride_head;
    s.kv.stride_seq = kv->stride_seq;
    s.kv.stride_page = kv->stride_page;
    s.kv.block_table = kv->block_table;
    s.kv.max_pages = kv->max_pages_per_seq;
    s.kv.page_tokens = kv->page_tokens;
    s.kv.n_kv_heads = kv->n_kv_heads;
    s.kv.head_dim = kv->head_dim;
    s.bv.seq_len = bv->seq_len;
    s.bv.vis_start = bv->vis_start;
    s.bv.vis_len = bv->vis_len;
    s.bv.max_seq_len = bv->max_seq_len;
    s.bv.max_vis_len = bv->max_vis_len;
    s.batch = bv->batch;
    s.n_q_heads = n_q_heads;
    s.dtype = kv->dtype;
    s.paged = kv->page_tokens > 0;
    // The MFMA kernels read 16-byte vectors: every cache row must start 16-byte aligned.
    auto a16 = [](const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; };
    const bool aligned = a16(kv->k) && a16(kv->v) && kv->stride_token % 8 == 0 &&
                         kv->stride_head % 8 == 0 && kv->stride_seq % 8 == 0 && kv->stride_page % 8 == 0;
    s.fast = kv->dtype == FASTOCR_BF16 && (kv->head_dim == 128 || kv->head_dim == 64) && n_q_heads / kv->n_kv_heads <= 16 && aligned;
    const int64_t esz = kv->dtype == FASTOCR_BF16 ? 2 : 4;
    auto m16 = [&](int64_t elems) { return (elems * esz) % 16 == 0; };
    s.vec16 = a16(kv->k) && a16(kv->v) && m16(kv->stride_token) && m16(kv->stride_head) && m16(kv->stride_seq) &&
              m16(kv->stride_page) && m16(kv->head_dim);
    s.fast32 = kv->dtype == FASTOCR_F32 && (kv->head_dim == 128 || kv->head_dim == 64) && n_q_heads / kv->n_kv_heads <= 16 && s.vec16;
    return s;
}

static bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Number of position ranges per (sequence, kv head): enough workgroups to fill the chip a few
// times over, never less than one tile per wave.  A pure function of the host-side shape so
// that the workspace query and the launch agree.
// Pruned attention as partials over four-wave workgroups of one tile per wave: the finest cut
// choose_splits ever makes of a short list.  *fits: such a cut leaves at most one workgroup per compute
// unit (only then is it taken).
static int finest_splits(const Shape &s, int max_positions, bool *fits = nullptr)
{
    const int streams = s.batch * s.kv.n_kv_heads;
    const int ntile = (max_positions + 31) / 32;
    const int by_work = (ntile + 3) / 4;
    const int most = streams > 0 ? plan_cu_count() / streams : 1;
    if (fits) *fits = by_work <= most;
    const int n = by_work < most ? by_work : most;
    return n < 1 ? 1 : n;
}

// Ranges per stream of the fp64 matrix-core kernels: two workgroups of four waves per compute unit, rounded down (see
// partial_rows).  Where that leaves at most 1.7 workgroups per compute unit, some hold two and the others one, with half
// the loads in flight; with one query head per kv head, where the kernels are bound by bytes and the plain kernels
// read no row twice either, a finer cut evens that out (head_dim 128, caches too large for the last-level cache, us: 264 streams
// of 700 tokens, 1 / 3 ranges, scoring 56.2 / 46.5, dense attention 60.3 / 51.2; 384 of 1700, 124.7 / 104.8, 141.0 / 127.6;
// 192 of 1700, 2 / 4 ranges, 65.3 / 55.6, 77.9 / 65.6; from 448 streams on one range is as good or better: 131.4 / 126.7, 141.7 / 148.7).
// A range keeps two blocks of 64 tokens (scoring, which ends in a second launch anyway: one and a half): 384 streams of 280, dense
// attention 31.0 / 35.4, 264 of them, scoring 33.2 / 30.7.
static int f32_ranges(int op, const Shape &s, int num_cu, int blocks)
{
    const int64_t streams = std::max<int64_t>(1, (int64_t)s.batch * s.kv.n_kv_heads);
    const int n = (int)std::max<int64_t>(1, 2 * num_cu / streams);
    const int64_t filled = n * streams;
    const bool uneven = s.n_q_heads == s.kv.n_kv_heads && filled > num_cu && 10 * filled <= 17 * num_cu;
    const int finer = n + std::max(2, n);
    return uneven && 2 * blocks >= (op == FASTOCR_OP_FOCAL_SCORE ? 3 : 4) * finer ? finer : n;
}

// Dense attention of bf16 caches over a list so short that one eight-wave workgroup per stream, which writes the output itself, is
// done before partials and their merge would be: a launch less against one compute unit's load path (us, ranges and merge / one:
// head_dim 128, 4 streams of 8 / 12 / 16 tiles 7.0 / 5.0, 7.0 / 5.9, 7.2 / 7.7; 32 streams 7.7 / 6.0, 7.7 / 7.2, 7.8 / 8.5; 64 of
// 12 / 16 / 20 8.3 / 7.5, 8.9 / 8.9, 9.7 / 10.2; 96 of 16 / 24 / 32 10.5 / 9.3, 12.0 / 11.9, 14.0 / 14.9; 128 of 16 / 32 / 40
// 12.1 / 9.6, 17.3 / 16.4, 19.0 / 18.3, but lists of 5 .. 40 14.8 / 15.1; head_dim 64, 8 and 32 streams of 8 / 12 7.8 / 7.2,
// 7.9 / 8.0 and 8.1 / 7.6, 8.0 / 8.3; 128 of 16 / 24 9.9 / 9.3, 10.6 / 10.6).
static bool dense_in_one(const Shape &s, int ntile, int num_cu)
{
    const int streams = s.batch * s.kv.n_kv_heads;
    if (s.kv.head_dim == 64) return ntile <= (2 * streams >= num_cu ? 24 : 8);
    return ntile <= (2 * streams >= num_cu ? 32 : (8 * streams >= 3 * num_cu ? 24 : (4 * streams >= num_cu ? 16 : 12)));
}

// Ranges per stream of the bf16 streaming kernels (dense attention, scoring, kernels that park their logits): about one workgroup of four waves per
// compute unit, rounded down (see choose_splits), except where streams of unlike lengths -- the host knows the longest only -- or an uneven
// last round would leave compute units idle.  Measured in us, "equal": all sequences as long as the longest, "unlike": an eighth to all of that,
// the mean of three to five batches.
static int even_ranges(int op, const Shape &s, int ntile, int num_cu, bool parks)
{
    const int streams = s.batch * s.kv.n_kv_heads;
    if (streams < 1) return 1;
    int n = std::max(1, num_cu / streams);
    if (op == FASTOCR_OP_FOCAL_SCORE) {
        // Scoring holds half the loads per workgroup (no V): two workgroups per compute unit where a stream gets only a few ranges
        // (one / two per compute unit: head_dim 64, 96 streams of 4288 tokens 19.1 / 16.3, 144 of 1216 12.4 / 10.4; head_dim 128, 144 of 1192
        // 16.0 / 14.6, 16 of 4288 9.3 / 9.6), doubled while a range has more than 1024 tokens
        // (scoring in two launches, without / with the doubling, equal then unlike: 64/8 heads, 22 x 12000 141.8 / 120.5, 108.7 / 86.0; 28/4, 36 x 6000 54.8 / 53.7, 42.5 / 36.8;
        // head_dim 64, 64/8, 36 x 8000 104.5 / 80.6, 85.5 / 65.1; 8/1, 176 x 12000 158.4 / 136.6, 124.2 / 97.5)
        if (4 * streams > num_cu) n = std::max(1, 2 * num_cu / streams);
        while (ntile > 32 * n) n *= 2;
    }
    // A little more than a chip of streams, in kernels that leave partials anyway, in halves (one range / two, equal then unlike: 28/4 heads, 72 x 1000,
    // scoring 26.0 / 23.0, 20.3 / 18.4, focal layer 43.2 / 38.4, 34.2 / 26.7; 96 x 500, 17.0 / 15.9, 14.0 / 12.7, 28.5 / 28.3, 23.2 / 22.2;
    // short lists the other way: 72 x 200, layer 16.7 / 16.7, 14.7 / 15.4; and so do streams near two chips: head_dim 64, 32/8, 60 x 600, layer
    // 23.8 / 27.4)
    if ((parks || op == FASTOCR_OP_FOCAL_SCORE) && streams > num_cu && 2 * streams <= 3 * num_cu && ntile >= 16) n = std::max(n, 2);
    // Dense attention of half a chip of streams to a whole one: one range each leaves up to half of the compute units idle and lasts as long as the
    // longest sequence, two fill the chip unevenly.  Three or four, which fill two or three rounds, from the length on where unlike lists gain more
    // than equal ones lose (one / two / three or four ranges, equal then unlike; 64/8 heads: 17 x 2700 35.1 / 44.5 / 35.2, 31.1 / 30.0 / 27.9;
    // 17 x 12000 139 / 172 / 131, 120 / 92 / 94; 21 x 2700 38.1 / 46.3 / 42.1, 32.5 / 31.6 / 30.2; 21 x 6000 79.9 / 94.0 / 83.6, 66.0 / 63.4 / 57.0;
    // 22 x 6000 82.8 / 94.2 / 86.2, 66.4 / 66.6 / 57.1; 22 x 16900 226 / 249 / 227, 185 / 164 / 152; 28 x 12000 200 / 210 / 211, 147 / 150 / 148;
    // head_dim 64: 17 x 3300 25.1 / 33.0 / 26.5, 23.1 / 21.6 / 22.1; 17 x 6000 40.9 / 51.8 / 39.9, 37.4 / 35.0 / 33.0; and beyond three quarters of a
    // chip 31 x 16900 165.5 / 160.1, 118.4 / 110.8, where head_dim 128 takes 260 / 267, 199 / 192 at 26 x 16900)
    if (op == FASTOCR_OP_DENSE_DECODE_ATTN && !parks && 2 * streams > num_cu && streams <= num_cu) {
        if (4 * streams > 3 * num_cu) n = s.kv.head_dim == 64 && ntile >= 512 ? 2 : 1;
        else if (3 * streams > 2 * num_cu) n = ntile >= 384 ? 4 : 1;
        else if (5 * streams > 3 * num_cu) n = ntile >= 192 ? 3 : 1;
        else n = ntile >= (s.kv.head_dim == 64 ? 160 : 80) ? 3 : 1;
    }
    return n;
}

// replay: 0 / 1 = as if "graph_replay" were that, -1 = the tuning's value.  *partials (if given) is set
// when the choice only holds as partials in the workspace followed by the merge kernel.  parks: ranges of the kernel that parks its
// logits, which a second launch follows anyway.
static int choose_splits(int op, const Shape &s, int max_positions, bool *partials = nullptr, int replay = -1, bool parks = false)
{
    if (partials) *partials = false;
    if (replay < 0) replay = g_tune_graph_replay.load(std::memory_order_relaxed);
    const bool fast = s.fast;
    const int kNumCU = plan_cu_count();
    const int forced = g_tune_splits[op].load(std::memory_order_relaxed);
    const int tile = fast ? 32 : 64;
    const int waves_per_wg = fast ? 4 : 1;
    const int ntile = (max_positions + tile - 1) / tile;
    const int by_work = (ntile + waves_per_wg - 1) / waves_per_wg;
    int nsplit;
    if (forced > 0) {
        nsplit = forced;
    } else {
        const int streams = s.batch * (fast || s.fast32 ? s.kv.n_kv_heads : s.n_q_heads);
        // Measured on MI355X: the streaming kernels run best with about one workgroup per compute
        // unit (few, long, equally sized streams), the plain-FMA kernels with many small ones.
        const int target_wg = 8 * kNumCU;
        if (fast && op == FASTOCR_OP_SPARSE_DECODE_ATTN && g_tune_attn_merge.load(std::memory_order_relaxed)) {
            // pruned attention is short: one launch whose eight-wave workgroups fill the chip once,
            // the ranges of a stream merged inside the launch.  Up to 14 tiles one workgroup has the whole list
            // in flight at once (two tiles per wave) and a cut only adds the merge; beyond that a compute
            // unit's load path is the bound, and the ranges that leave a wave at most one tile win until four
            // of them no longer do (us per call with 1 / 2 / 3 / 4 ranges, 32 streams: 12 tiles 8.0 / 8.7 / 9.0 / 9.0,
            // 15 tiles 8.9 / 8.8 / 8.9 / 9.5, 20 tiles 10.5 / 10.0 / 9.0 / 9.6, 27 tiles 13.2 / 10.8 / 9.7 / 9.4,
            // 40 tiles 16.1 / 13.1 / 11.3 / 11.7, 52 tiles 20.2 / 14.9 / 12.6 / 11.7; 4, 24 and 128 streams
            // order alike)
            int n = kNumCU / (streams > 0 ? streams : 1);
            const int by_len = ntile <= 14 ? 1 : (ntile <= 16 ? 2 : (ntile <= 24 ? 3 : (ntile <= 32 || ntile >= 48 ? 4 : 3)));
            n = n < by_len ? n : by_len;
            n = n < 1 ? 1 : n;
            if (n == 1 || attn_merges_in_kernel(s, n)) {
                // A compute unit gathers rows at a few tens of GB/s, so a short list of few streams is
                // done sooner the more compute units share it -- but every range a stream is cut into
                // makes the in-launch merge wait longer for words to cross the chip (3 - 4 us against a
                // plain store of the partial).  Replayed from a graph, where the merge kernel starts
                // 0.4 us after the launch before it (eager: 2 - 3 us), partials over four-wave workgroups
                // of one tile per wave plus that kernel win as long as those workgroups find a compute
                // unit each (a captured step of 28 layers, single launches / fine cut: 296 / 291 us with 32 streams of
                // 15 tiles, 325 / 297 and 307 / 283 with 24 of 27, 371 / 292 and 354 / 280 with 8 of 47, 265 / 240
                // with 4 of 17; with 96 and 128 streams of 15 tiles, where they would not, an earlier form of
                // the kernel took 418 / 464 and 449 / 506 us, so those keep the single launch; eager the fine cut costs
                // 2 us per call).
                bool fits = false;
                const int fine = finest_splits(s, max_positions, &fits);
                if (replay == 1 && fits && fine > n) {
                    if (partials) *partials = true;
                    return fine;
                }
                return n;
            }
        }
        if (s.fast32) {
            nsplit = f32_ranges(op, s, kNumCU, by_work);
            // a list of up to two (head_dim 64: three) tiles per wave is not cut: the one launch then writes the output
            // itself (us uncut / cut, launched one by one and replayed from a graph: head_dim 128, 100 tokens 10.1 / 12.3 and 9.8 /
            // 9.2, 160 tokens -- three tiles, cut -- 12.8 / 12.3 and 12.8 / 9.4; head_dim 64, 160 tokens 9.8 / 12.5 and 8.0 / 7.6:
            // a replay would gain half a microsecond from a cut, single launches lose two, so the line is theirs for both)
            if (op != FASTOCR_OP_FOCAL_SCORE && by_work <= (s.kv.head_dim == 64 ? 3 : 2)) nsplit = 1;
        }
        // Dense attention of bf16 caches: rounded down, so that no compute unit holds two workgroups while others hold one (192 of
        // 256 compute units already draw what the memory delivers; us with the range count rounded up / down, merge included:
        // 28/4 heads, 12 x 1024 image tokens 12.5 / 11.0, 12 x 4096 26.3 / 21.6, 12 x 16384 81.6 / 64.7; 16/2 heads, 12 x 4096 17.5 / 14.4,
        // 12 x 16384 47.1 / 35.4; head_dim 64, 32/8 heads, 12 x 4096 28.9 / 22.1; 64/8, 11 x 2048 27.2 / 21.5, where five ranges, 440
        // workgroups, take 21.6).
        else if (fast) nsplit = even_ranges(op, s, ntile, kNumCU, parks);
        else nsplit = (target_wg + streams - 1) / (streams > 0 ? streams : 1);
        // pruned attention is short: when eight waves get at most eight tiles each, or at least half
        // a chip of streams exists, one eight-wave workgroup per stream writes the final output
        // itself (no partials, no merge kernel -- a second launch costs more than it saves here)
        if (fast && op == FASTOCR_OP_SPARSE_DECODE_ATTN && (2 * streams >= kNumCU || ntile <= 64)) nsplit = 1;
        if (fast && op == FASTOCR_OP_DENSE_DECODE_ATTN && !parks && dense_in_one(s, ntile, kNumCU)) nsplit = 1;
    }
    if (nsplit > by_work) nsplit = by_work;
    if (nsplit > 256) nsplit = 256;
    if (nsplit < 1) nsplit = 1;
    return nsplit;
}

// Partial rows (sequence, query head, range) to size a workspace for: the most that a call with this many sequences or fewer, as long or
// shorter, leaves (a call's own count goes up and down with both, by the rounding of its range count).
// bf16 on the matrix cores: ranges of at least four tiles that fill the chip at most once (scoring, from a quarter of a chip of streams on:
// twice), or one range per stream.
// fp32 on the matrix cores (see f32_ranges): at most 2 CU workgroups with a row per query head of their group, or with one
// head per group 3.4 CU of them, or three ranges of up to 1.7 CU streams, or one range per sequence.  That is at most 8192
// rows of 256 CUs and 16 heads, 4.3 MB at head_dim 128, unless the batch itself has more, so every shape whose single
// ranges fit the static scratch is served from it.
static size_t partial_rows(int op, const Shape &s, int max_positions, int nsplit, bool parks = false)
{
    const size_t heads = (size_t)s.batch * s.n_q_heads;
    if (!(s.fast || s.fast32) || g_tune_splits[op].load(std::memory_order_relaxed) > 0) return heads * nsplit;
    const size_t cus = (size_t)plan_cu_count(), Hkv = (size_t)s.kv.n_kv_heads;
    if (s.fast) {
        const size_t streams = s.batch * Hkv, tiles = (size_t)(max_positions + 31) / 32, by_work = std::min<size_t>(256, std::max<size_t>(1, (tiles + 3) / 4));
        size_t filled = std::max(streams, cus);                           // see even_ranges
        if (op == FASTOCR_OP_FOCAL_SCORE) filled = std::max({filled, 4 * streams > cus ? 2 * cus : 0, streams * (tiles / 16)});
        if (op == FASTOCR_OP_FOCAL_SCORE || parks) { if (streams > cus) filled = std::max(filled, std::min(2 * streams, 3 * cus)); }
        else if (op == FASTOCR_OP_DENSE_DECODE_ATTN && 2 * streams > cus) filled = std::max(filled, 3 * cus);
        return s.n_q_heads / Hkv * std::min(streams * by_work, filled);
    }
    const size_t by_work = (size_t)std::min(256, std::max(1, (max_positions + 63) / 64));
    size_t filled = 2 * cus / Hkv;                                        // sequences times ranges
    if ((size_t)s.n_q_heads == Hkv) {
        filled = 34 * cus / 10 / Hkv;
        if (s.batch * Hkv > cus) filled = std::max(filled, 3 * std::min((size_t)s.batch, 17 * cus / 10 / Hkv));
    }
    filled *= (size_t)s.n_q_heads;
    return std::min(heads * by_work, std::max(heads, filled));
}

// Upper bound of the positions a pruned-attention call attends: all text plus kmax image tokens
// (kmax <= 0: unknown, the whole sequence).
static int sparse_positions(const fastocr_batch_view *bv, int64_t kmax)
{
    if (kmax <= 0 || kmax >= bv->max_vis_len) return bv->max_seq_len;
    return bv->max_seq_len - bv->max_vis_len + (int)kmax;
}

static size_t round256(size_t x) { return (x + 255) / 256 * 256; }

}  // namespace fastocr

using namespace fastocr;

extern "C" {

int64_t fastocr_keep_count(int64_t n_visual, double tau)
{
    if (n_visual <= 0 || !(tau > 0.0)) return 0;
    double x = ceil(tau * (double)n_visual - 1e-9);
    if (x < 0.0) x = 0.0;
    if (x > (double)n_visual) x = (double)n_visual;
    return (int64_t)x;
}

size_t fastocr_workspace_bytes(int op, const fastocr_kv_view *kv, const fastocr_batch_view *bv,
                               int n_q_heads, int64_t kmax)
{
    if (op == FASTOCR_OP_TOPK_FIXATION) {
        if (!bv || bv->batch < 0 || bv->max_vis_len < 0) return 0;
        return round256(topk_workspace_bytes(bv->batch, bv->max_vis_len));
    }
    if (op == FASTOCR_OP_FOCAL_SCORE_TOPK || op == FASTOCR_OP_FOCAL_ATTN_SCORE_TOPK) {
        // the fused launch, or the two separate calls one after the other in the same buffer
        const size_t a = fastocr_workspace_bytes(op == FASTOCR_OP_FOCAL_SCORE_TOPK ? FASTOCR_OP_FOCAL_SCORE : FASTOCR_OP_FOCAL_ATTN_SCORE,
                                                 kv, bv, n_q_heads, 0);
        const size_t b = fastocr_workspace_bytes(FASTOCR_OP_TOPK_FIXATION, kv, bv, n_q_heads, kmax);
        return a == 0 ? 0 : (a > b ? a : b);
    }
    if (op < 0 || op > FASTOCR_OP_FOCAL_ATTN_SCORE) return 0;
    if (check_views(kv, bv, n_q_heads) != FASTOCR_OK) return 0;
    Shape s = make_shape(kv, bv, n_q_heads);
    if (op == FASTOCR_OP_FOCAL_ATTN_SCORE) {
        // the one-pass kernel, or the two separate calls one after the other in the same buffer
        size_t need = fastocr_workspace_bytes(FASTOCR_OP_FOCAL_SCORE, kv, bv, n_q_heads, 0);
        const size_t dense = fastocr_workspace_bytes(FASTOCR_OP_DENSE_DECODE_ATTN, kv, bv, n_q_heads, 0);
        need = need > dense ? need : dense;
        if (s.fast32) {
            const int nsplit = choose_splits(FASTOCR_OP_DENSE_DECODE_ATTN, s, bv->max_seq_len);
            const size_t rows = partial_rows(FASTOCR_OP_DENSE_DECODE_ATTN, s, bv->max_seq_len, nsplit);
            const size_t one = round256(focal_f32_workspace_bytes(s, rows) + 256);
            need = need > one ? need : one;
        }
        if (parks_by_head(s)) {
            const int nsplit = choose_splits(FASTOCR_OP_DENSE_DECODE_ATTN, s, bv->max_seq_len, nullptr, -1, true);
            const size_t rows = partial_rows(FASTOCR_OP_DENSE_DECODE_ATTN, s, bv->max_seq_len, nsplit, true);
            need = std::max(need, round256(focal_parked_workspace_bytes(s, rows) + 256));
        }
        const size_t fused = focal_fused_workspace_bytes(s, plan_cu_count());
        return fused > 0 ? std::max(need, round256(fused + 256)) : need;
    }
    // (pruned attention: whatever "graph_replay" asks for, and a size taken with a larger kmax, or none, also covers)
    const int positions = op == FASTOCR_OP_SPARSE_DECODE_ATTN ? sparse_positions(bv, kmax) : bv->max_seq_len;
    const int nsplit = choose_splits(op, s, positions, nullptr, 0);
    if (op == FASTOCR_OP_FOCAL_SCORE) {
        // sized for either scoring path, so that the choice can be made at launch
        size_t need = score_workspace_bytes(s, partial_rows(op, s, positions, nsplit));
        ResidentPlan rp;
        if (resident_plan(s, plan_cu_count(), &rp)) need = need > resident_workspace_bytes(s, rp) ? need : resident_workspace_bytes(s, rp);
        return round256(need + 256);
    }
    return round256(attn_workspace_bytes(s, partial_rows(op, s, positions, nsplit)) + 256);
}

static int check_ws(const void *ws, size_t ws_bytes, size_t need)
{
    if (need == 0) return FASTOCR_OK;
    if (!ws || (reinterpret_cast<uintptr_t>(ws) & 255u) != 0 || ws_bytes < need) return FASTOCR_EWORKSPACE;
    return FASTOCR_OK;
}

static int check_qo(const fastocr_kv_view *kv, const void *q, const void *out, float scale)
{
    if (!q || !isfinite(scale)) return FASTOCR_EINVAL;
    if (!aligned16(q) || (out && !aligned16(out))) return FASTOCR_EINVAL;
    (void)kv;
    return FASTOCR_OK;
}

// The register-resident kernels (scoring alone, or fused with the dense output) read K and V and write scores, but their
// workgroups exchange statistics across the grid and finish in a chain of steps that nothing hides: 9 - 20 us whatever the size,
// and more in a ragged batch, whose ranges every wave works out for itself.  Kernels that park the logits in memory
// for a second launch have no such chain and pay for the logits' bytes, written into a read stream and read back.  So the library
// parks up to this many bytes of logits (batch x query heads x longest sequence x 4; us, register-resident / parked; caches too
// large for the last-level cache where there is room):
//   scoring            28/4 heads: batch 1, 4096 image tokens 11.9 / 8.7, 4 x 4096 15.6 / 9.3, 12 x 4096 (5.8 MB) 17.7 / 15.7, 8 x 8192 (7.5) 19.9 / 19.9,
//                      12 x 8192 (11.3) 24.4 / 27.2; 64/8 heads 12 x 2048 (6.9) 18.0 / 17.0, 8 x 4096 (8.8) 20.3 / 21.0.  Sequences of equal length
//                      lose from about 5.5 MiB on, most with many short ones (64/8, 17 x 1500 18.4 / 19.7; 32/8, 36 x 1500 24.2 / 27.9; of 503 shapes
//                      below the limit 17 by more than 3 %, at most 16 %); lengths from an eighth of the longest to all of it gain up to
//                      the limit and beyond (28/4, 16 x 4000 22.0 / 16.5; 64/8, 22 x 1000 19.4 / 13.8; of 468 none loses, on the mean -25 % at
//                      5.5 - 7 MiB).  The host knows the longest sequence only; a decode batch seldom has equal ones
//   layer and top-k    28/4: 1 x 4096 21.5 / 14.8, 12 x 4096 34.5 / 31.3, 8 x 8192 40.2 / 39.2, 12 x 6200 (8.03 MiB) 43.6 / 42.3, 12 x 8192 50.0 / 52.1;
//                      64/8: 16 x 2048 (8.25) 44.2 / 41.2; 12/2: 24 x 7300 (8.09) 45.7 / 47.1, 24 x 8192 51.6 / 52.4; head_dim 64, 64/8: 16 x 2100 (8.45)
//                      31.7 / 32.5: these last rows set the limit
//   layer alone        gains further up (28/4: 12 x 6200 40.9 / 35.4, 12 x 8192 47.4 / 45.0, 16 x 8192 (15.0) 59.5 / 59.3; 64/8: 16 x 2048 39.2 / 34.1,
//                      12 x 4096 (13.2) 48.6 / 49.4; head_dim 64, 64/8: 12 x 4096 32.2 / 32.7), but has the form, and so the bits, of the call with its top-k
//   ragged and paged   28/4, 12 sequences of up to 5000: scoring 25.4 / 16.7, layer and top-k 42.4 / 32.0
//   mostly text        28/4, 12 x 200 image tokens and 5000 of text: scoring 33.3 / 16.7, layer 63.4 / 27.7; 1 x 64 and 16000: 280 / 9.5, 559 / 13.3
// Where the single kernel is not to be had (head counts, a stream without a slot, a process that distrusts the exchange) a layer parks at every
// size, instead of dense attention and then scoring: 28/4, 12 x 8192 80.5 / 46.2; 64/8, 16 x 16384 283 / 231; 96/8, 16 x 16384 312 / 251.
constexpr int64_t kParkScore = 7 << 20, kParkLayer = 8 << 20;

static bool select_inside() { return g_tune_select_fused.load(std::memory_order_relaxed) != 0; }

static bool parks(int mode, const Shape &s, int64_t limit)
{
    return mode == 1 && parks_by_head(s) &&
           (int64_t)s.batch * s.n_q_heads * s.bv.max_seq_len * (int64_t)sizeof(float) <= limit;
}

// mode: the tuning value (0 never, 1 the library's choice, 2 whenever the shape fits).  The
// library's own choice also requires that no wave of a single-launch form has ever given up
// waiting in this process: a launch that cannot have the chip to itself is not tried twice.
// On success *slot is the call's exchange slot.
static bool use_resident(int kind, int mode, const Shape &s, ResidentPlan *rp, hipStream_t stream, int *slot, uint32_t **flag)
{
    const int cus = plan_cu_count();
    if (mode == 0 || !resident_plan(s, cus, rp)) return false;
    if (rp->nranges * s.batch > cus) return false;
    if (mode != 2 && !exchange_trusted()) return false;
    *slot = exchange_slot(kind, stream, flag);
    return *slot >= 0;
}

static int check_topk_args(const float *scores, const fastocr_batch_view *bv, double tau, const int32_t *prev_idx,
                           const int32_t *prev_cnt, int32_t *sel_idx, int32_t *sel_cnt, int64_t kmax)
{
    if (!bv || bv->batch < 0 || bv->max_vis_len < 0 || bv->max_seq_len < 0) return FASTOCR_EINVAL;
    if (bv->max_vis_len > bv->max_seq_len) return FASTOCR_EINVAL;
    if (bv->batch > 65535) return FASTOCR_EUNSUPPORTED;
    if (!(tau >= 0.0 && tau <= 1.0)) return FASTOCR_EINVAL;
    if (bv->batch > 0 && (!bv->seq_len || !bv->vis_start || !bv->vis_len)) return FASTOCR_EINVAL;
    if (!sel_idx || !sel_cnt) return FASTOCR_EINVAL;
    if (!scores && bv->max_vis_len > 0 && bv->batch > 0) return FASTOCR_EINVAL;
    if ((prev_idx == nullptr) != (prev_cnt == nullptr)) return FASTOCR_EINVAL;
    if (kmax < 1 || kmax < fastocr_keep_count(bv->max_vis_len, tau)) return FASTOCR_EINVAL;
    return FASTOCR_OK;
}

// Scoring, optionally with the top-k inside the same launch (select != nullptr).  *fused tells the
// caller whether the select ran inside the launch; if not, it still has to be called.
static int focal_score_impl(const fastocr_kv_view *kv, const fastocr_batch_view *bv, const void *q,
                            int n_q_heads, float scale, float *scores, float *lse, float *img_mass,
                            void *ws, size_t ws_bytes, void *hip_stream, const SelectArgs *select, bool *fused)
{
    if (fused) *fused = false;
    int rc = check_views(kv, bv, n_q_heads);
    if (rc != FASTOCR_OK) return rc;
    rc = check_qo(kv, q, nullptr, scale);
    if (rc != FASTOCR_OK) return rc;
    if (!scores && bv->max_vis_len > 0 && bv->batch > 0) return FASTOCR_EINVAL;
    const size_t need = fastocr_workspace_bytes(FASTOCR_OP_FOCAL_SCORE, kv, bv, n_q_heads, 0);
    rc = check_ws(ws, ws_bytes, need);
    if (rc != FASTOCR_OK) return rc;
    if (bv->batch == 0) return FASTOCR_OK;
    Shape s = make_shape(kv, bv, n_q_heads);
    const int nsplit = choose_splits(FASTOCR_OP_FOCAL_SCORE, s, bv->max_seq_len);
    ResidentPlan rp;
    hipError_t e;
    int slot = -1;
    uint32_t *flag = nullptr;
    const int mode = g_tune_score_resident.load(std::memory_order_relaxed);
    const bool fuse = select && select_inside() && resident_select_fits(s);
    const bool park = parks(mode, s, kParkScore);
    if (!park && use_resident(EX_SCORE, mode, s, &rp, (hipStream_t)hip_stream, &slot, &flag)) {
        e = launch_score_resident(s, rp, slot, flag, q, scale, scores, lse, img_mass, ws, (hipStream_t)hip_stream, fuse ? select : nullptr);
        if (fused) *fused = fuse;
    } else {
        const bool selects = park && fuse;
        e = launch_score(s, q, scale, scores, lse, img_mass, ws, nsplit, (hipStream_t)hip_stream, selects ? select : nullptr);
        if (fused) *fused = selects;
    }
    return e == hipSuccess ? FASTOCR_OK : FASTOCR_EHIP;
}

int fastocr_focal_score(const fastocr_kv_view *kv, const fastocr_batch_view *bv, const void *q,
                        int n_q_heads, float scale, float *scores, float *lse, float *img_mass,
                        void *ws, size_t ws_bytes, void *hip_stream)
{
    return focal_score_impl(kv, bv, q, n_q_heads, scale, scores, lse, img_mass, ws, ws_bytes, hip_stream, nullptr, nullptr);
}

int fastocr_focal_score_topk(const fastocr_kv_view *kv, const fastocr_batch_view *bv, const void *q,
                             int n_q_heads, float scale, double tau, const int32_t *prev_idx,
                             const int32_t *prev_cnt, int32_t *sel_idx, int32_t *sel_cnt, int64_t kmax,
                             float *scores, float *lse, float *img_mass, void *ws, size_t ws_bytes,
                             void *hip_stream)
{
    int rc = check_topk_args(scores, bv, tau, prev_idx, prev_cnt, sel_idx, sel_cnt, kmax);
    if (rc != FASTOCR_OK) return rc;
    const size_t need = fastocr_workspace_bytes(FASTOCR_OP_FOCAL_SCORE_TOPK, kv, bv, n_q_heads, kmax);
    if (need == 0) return check_views(kv, bv, n_q_heads) != FASTOCR_OK ? check_views(kv, bv, n_q_heads) : FASTOCR_EINVAL;
    rc = check_ws(ws, ws_bytes, need);
    if (rc != FASTOCR_OK) return rc;
    const SelectArgs sa{tau, prev_idx, prev_cnt, sel_idx, sel_cnt, kmax};
    bool fused = false;
    rc = focal_score_impl(kv, bv, q, n_q_heads, scale, scores, lse, img_mass, ws, ws_bytes, hip_stream, &sa, &fused);
    if (rc != FASTOCR_OK || fused) return rc;
    return fastocr_topk_fixation(scores, bv, tau, prev_idx, prev_cnt, sel_idx, sel_cnt, kmax, ws, ws_bytes, hip_stream);
}

int fastocr_topk_fixation(const float *scores, const fastocr_batch_view *bv, double tau,
                          const int32_t *prev_idx, const int32_t *prev_cnt, int32_t *sel_idx,
                          int32_t *sel_cnt, int64_t kmax, void *ws, size_t ws_bytes, void *hip_stream)
{
    const int rc0 = check_topk_args(scores, bv, tau, prev_idx, prev_cnt, sel_idx, sel_cnt, kmax);
    if (rc0 != FASTOCR_OK) return rc0;
    const size_t need = fastocr_workspace_bytes(FASTOCR_OP_TOPK_FIXATION, nullptr, bv, 0, kmax);
    int rc = check_ws(ws, ws_bytes, need);
    if (rc != FASTOCR_OK) return rc;
    if (bv->batch == 0) return FASTOCR_OK;
    BatchDev bd{bv->seq_len, bv->vis_start, bv->vis_len, bv->max_seq_len, bv->max_vis_len};
    hipError_t e = launch_topk(scores, bd, bv->batch, tau, prev_idx, prev_cnt, sel_idx, sel_cnt, kmax,
                               ws, (hipStream_t)hip_stream);
    return e == hipSuccess ? FASTOCR_OK : FASTOCR_EHIP;
}

static int attn_common(int op, const fastocr_kv_view *kv, const fastocr_batch_view *bv, const void *q,
                       int n_q_heads, float scale, const int32_t *sel_idx, const int32_t *sel_cnt,
                       int64_t kmax, void *out, float *lse, void *ws, size_t ws_bytes, void *hip_stream,
                       bool static_ws = false)
{
    int rc = check_views(kv, bv, n_q_heads);
    if (rc != FASTOCR_OK) return rc;
    if (!out) return FASTOCR_EINVAL;
    rc = check_qo(kv, q, out, scale);
    if (rc != FASTOCR_OK) return rc;
    if (op == FASTOCR_OP_SPARSE_DECODE_ATTN && (!sel_idx || !sel_cnt || kmax < 1)) return FASTOCR_EINVAL;
    const size_t need = fastocr_workspace_bytes(op, kv, bv, n_q_heads, kmax);
    if (static_ws) {
        // the library's own buffer: a shape that needs more than it holds is refused before any GPU call
        if (need > (size_t)FASTOCR_STATIC_SCRATCH_BYTES) return FASTOCR_ETOOLARGE;
        if (bv->batch == 0) return FASTOCR_OK;
        ws = static_scratch_ptr();
        ws_bytes = FASTOCR_STATIC_SCRATCH_BYTES;
        if (!ws) return FASTOCR_EHIP;
    }
    rc = check_ws(ws, ws_bytes, need);
    if (rc != FASTOCR_OK) return rc;
    if (bv->batch == 0) return FASTOCR_OK;
    Shape s = make_shape(kv, bv, n_q_heads);
    bool partials = false;
    const int nsplit = choose_splits(op, s, op == FASTOCR_OP_SPARSE_DECODE_ATTN ? sparse_positions(bv, kmax) : bv->max_seq_len, &partials);
    // the ranges of a stream merged inside the launch: when asked for, the shape fits, the stream has
    // an exchange slot and no such wait has ever been given up in this process (the range count
    // does not depend on the last two, so the workspace the caller sized always covers the
    // separate merge kernel)
    const int mode = g_tune_attn_merge.load(std::memory_order_relaxed);
    int merge_slot = -1;
    uint32_t *flag = nullptr;
    // (never for the static-workspace entry point: the first in-launch merge on a device allocates
    // the pinned "gave up" word)
    if (!static_ws && !partials && ((op == FASTOCR_OP_SPARSE_DECODE_ATTN && mode != 0) || mode == 2) && attn_merges_in_kernel(s, nsplit)) {
        if (exchange_trusted()) merge_slot = exchange_slot(EX_MERGE, (hipStream_t)hip_stream, &flag);
        if (merge_slot < 0) merge_slot = kNoMergeSlot;
    }
    hipError_t e = launch_attn(s, q, scale, sel_idx, sel_cnt, kmax, out, lse, ws, nsplit, merge_slot, flag, (hipStream_t)hip_stream);
    return e == hipSuccess ? FASTOCR_OK : FASTOCR_EHIP;
}

int fastocr_sparse_decode_attn(const fastocr_kv_view *kv, const fastocr_batch_view *bv, const void *q,
                               int n_q_heads, float scale, const int32_t *sel_idx, const int32_t *sel_cnt,
                               int64_t kmax, void *out, void *ws, size_t ws_bytes, void *hip_stream)
{
    return attn_common(FASTOCR_OP_SPARSE_DECODE_ATTN, kv, bv, q, n_q_heads, scale, sel_idx, sel_cnt, kmax,
                       out, nullptr, ws, ws_bytes, hip_stream);
}

// Whether two layers' caches differ in their places alone.
static bool alike(const fastocr_kv_view &a, const fastocr_kv_view &b)
{
    return a.dtype == b.dtype && a.n_kv_heads == b.n_kv_heads && a.head_dim == b.head_dim && a.stride_token == b.stride_token &&
           a.stride_head == b.stride_head && a.stride_seq == b.stride_seq && a.page_tokens == b.page_tokens &&
           a.stride_page == b.stride_page && a.max_pages_per_seq == b.max_pages_per_seq;
}

// Layers one after the other read and write in their order: no output may lie in anything that is read by the layers (its own query apart), nor in another
// output.  (The pages of a paged cache are not looked at: how far its pool reaches is not known here.)
static bool layers_apart(int n, const fastocr_kv_view *kv, const fastocr_batch_view *bv, const void *const *q, int n_q_heads,
                         const int32_t *sel_idx, const int32_t *sel_cnt, int64_t kmax, void *const *out)
{
    const int64_t B = bv->batch, es = kv[0].dtype == FASTOCR_BF16 ? 2 : 4, row = (int64_t)kv[0].head_dim * es, io = B * n_q_heads * row;
    Outputs<kLayerSet> outs;
    Span spans[kLayerSet];
    for (int i = 0; i < n; ++i) spans[i] = span_of(out[i], io);
    if (!outs.set(spans, n)) return false;
    for (const int32_t *p : {bv->seq_len, bv->vis_start, bv->vis_len, sel_cnt})
        if (!outs.apart(span_of(p, B * 4), -1)) return false;
    if (!outs.apart(span_of(sel_idx, B * kmax * 4), -1)) return false;
    const uint64_t last = (uint64_t)(B - 1) * kv[0].stride_seq + (uint64_t)(kv[0].n_kv_heads - 1) * kv[0].stride_head +
                          (uint64_t)std::max(bv->max_seq_len - 1, 0) * kv[0].stride_token;          // the farthest row
    const int64_t cache = (int64_t)(last * es) + row;
    for (int i = 0; i < n; ++i) {
        if (!outs.apart(span_of(q[i], io), i)) return false;
        if (kv[i].page_tokens > 0) {
            if (!outs.apart(span_of(kv[i].block_table, B * kv[i].max_pages_per_seq * 4), -1)) return false;
        } else if (!outs.apart(span_of(kv[i].k, cache), -1) || !outs.apart(span_of(kv[i].v, cache), -1)) {
            return false;
        }
    }
    return true;
}

int fastocr_sparse_decode_attn_layers(int n_layers, const fastocr_kv_view *kv, const fastocr_batch_view *bv, const void *const *q,
                                      int n_q_heads, float scale, const int32_t *sel_idx, const int32_t *sel_cnt, int64_t kmax,
                                      void *const *out, void *ws, size_t ws_bytes, void *hip_stream)
{
    if (n_layers < 0 || (n_layers > 0 && (!kv || !q || !out))) return FASTOCR_EINVAL;
    bool together = n_layers > 1;
    for (int l = 0; l < n_layers; ++l) {
        int rc = check_views(&kv[l], bv, n_q_heads);
        if (rc != FASTOCR_OK) return rc;
        if (!out[l] || !sel_idx || !sel_cnt || kmax < 1) return FASTOCR_EINVAL;
        rc = check_qo(&kv[l], q[l], out[l], scale);
        if (rc != FASTOCR_OK) return rc;
        rc = check_ws(ws, ws_bytes, fastocr_workspace_bytes(FASTOCR_OP_SPARSE_DECODE_ATTN, &kv[l], bv, n_q_heads, kmax));
        if (rc != FASTOCR_OK) return rc;
        together = together && alike(kv[0], kv[l]) && make_shape(&kv[l], bv, n_q_heads).fast;
    }
    if (n_layers == 0 || bv->batch == 0) return FASTOCR_OK;
    together = together && g_tune_attn_merge.load(std::memory_order_relaxed) != 0 &&
               g_tune_splits[FASTOCR_OP_SPARSE_DECODE_ATTN].load(std::memory_order_relaxed) == 0;
    auto one_by_one = [&](int from, int n) {
        for (int l = from; l < from + n; ++l) {
            const int rc = fastocr_sparse_decode_attn(&kv[l], bv, q[l], n_q_heads, scale, sel_idx, sel_cnt, kmax, out[l], ws, ws_bytes, hip_stream);
            if (rc != FASTOCR_OK) return rc;
        }
        return (int)FASTOCR_OK;
    };
    for (int l = 0, n; l < n_layers; l += n) {
        n = together ? std::min({kLayerSet, n_layers - l, 65535 / bv->batch}) : 1;
        if (n < 2 || !layers_apart(n, kv + l, bv, q + l, n_q_heads, sel_idx, sel_cnt, kmax, out + l)) {
            const int rc = one_by_one(l, n);
            if (rc != FASTOCR_OK) return rc;
            continue;
        }
        const Shape s = make_shape(&kv[l], bv, n_q_heads);
        // Ranges as for that many sequences, where they merge inside the launch.  Together is the faster side from 2 layers and 8 streams each on (us, together / one
        // by one, equal lists: 28/4 heads, 2 layers of 32 streams, 840 rows 10.1 / 18.1; 5 of 128, 1600 rows 83 / 109; 3 of 256, 3200 rows 189 / 197; 64/8 and head_dim
        // 64 alike; 135 shapes of 420 to 3200 rows, equal and unlike), but for lists of 100 tiles whose streams are a little more than a chip (2 layers of 132 to 160, 3 of 96):
        // equal lists 91 - 96 / 84 - 89, where unlike ones still gain, 66 - 70 / 74 - 78, and the host knows the longest only.
        Shape all = s;
        all.batch = s.batch * n;
        const int positions = sparse_positions(bv, kmax);
        int nsplit = choose_splits(FASTOCR_OP_SPARSE_DECODE_ATTN, all, positions, nullptr, 0), slot = -1;
        uint32_t *flag = nullptr;
        if (nsplit > 1 && !attn_merges_in_kernel(all, nsplit)) {
            // Few streams of long lists in groups of more heads than that merge takes (9 to 16 per kv head, beyond 64 tiles): one range per
            // stream lasts as long as its list, whatever the layers; their own calls, cut into many ranges and merged by a launch, add up.
            // Measured in us, together / one by one, batch 1 to 8: 69 tiles, 2 layers 17.5 - 25.7 / 15.9 - 23.1, 3 22.2 - 26.4 / 24.4 - 34.4,
            // 6 23.5 - 28.9 / 48.8 - 69.9; 125 tiles, 3 36.9 - 43.2 / 25.0 - 38.0, 6 38.7 - 47.5 / 49.7 - 78.1; 250 tiles, 6 71 - 90 / 63 - 112, 13
            // 76 - 92 / 135 - 169
            if ((positions + 31) / 32 > 24 * n) {
                const int rc = one_by_one(l, n);
                if (rc != FASTOCR_OK) return rc;
                continue;
            }
            nsplit = 1;
        } else if (nsplit > 1) {
            if (exchange_trusted()) slot = exchange_slot(EX_MERGE, (hipStream_t)hip_stream, &flag);
            if (slot < 0) {
                // The same ranges as each layer's partials and a merge launch (kNoMergeSlot): the outputs' bits do not depend on how many streams
                // are in use.  (ws holds them: a layer's own streams times nsplit are at most a chip, and nsplit at most a range per four tiles.)
                for (int i = l; i < l + n; ++i) {
                    const hipError_t e = launch_attn(make_shape(&kv[i], bv, n_q_heads), q[i], scale, sel_idx, sel_cnt, kmax, out[i], nullptr, ws,
                                                     nsplit, kNoMergeSlot, nullptr, (hipStream_t)hip_stream);
                    if (e != hipSuccess) return FASTOCR_EHIP;
                }
                continue;
            }
        }
        LayerPtrs at[kLayerSet];
        for (int i = 0; i < n; ++i) at[i] = LayerPtrs{kv[l + i].k, kv[l + i].v, q[l + i], out[l + i], kv[l + i].block_table};
        const hipError_t e = launch_attn_layers(s, n, at, scale, sel_idx, sel_cnt, kmax, nsplit, slot < 0 ? 0 : slot, flag, (hipStream_t)hip_stream);
        if (e != hipSuccess) return FASTOCR_EHIP;
    }
    return FASTOCR_OK;
}

int fastocr_dense_decode_attn(const fastocr_kv_view *kv, const fastocr_batch_view *bv, const void *q,
                              int n_q_heads, float scale, void *out, float *lse, void *ws, size_t ws_bytes,
                              void *hip_stream)
{
    return attn_common(FASTOCR_OP_DENSE_DECODE_ATTN, kv, bv, q, n_q_heads, scale, nullptr, nullptr, 0,
                       out, lse, ws, ws_bytes, hip_stream);
}

int fastocr_dense_decode_attn_static(const fastocr_kv_view *kv, const fastocr_batch_view *bv, const void *q,
                                     int n_q_heads, float scale, void *out, float *lse, void *hip_stream)
{
    return attn_common(FASTOCR_OP_DENSE_DECODE_ATTN, kv, bv, q, n_q_heads, scale, nullptr, nullptr, 0,
                       out, lse, nullptr, 0, hip_stream, /*static_ws=*/true);
}

// Whether a focal layer's top-k and the merge of its output's partials share a launch.  They do as long as the merges, each
// a workgroup of that launch's 1024 threads, pass through the chip in two or three rounds; in workgroups of 256 threads
// and a launch of their own (3 us) they are done sooner beyond that (us per call, shared / apart, 1024 image tokens:
// head_dim 128, 896 merges 32.4 / 34.6, 1024 35.2 / 36.0, 1680 43.9 / 42.2, 2048 49.1 / 46.3; head_dim 64, 1024 26.4 / 27.2,
// 1680 31.9 / 30.3, 2048 35.0 / 32.2, 6400 77.8 / 60.0).
static bool merge_shares_topk(const Shape &s)
{
    return topk_takes_combine(s.bv.max_vis_len, s.kv.head_dim) && (int64_t)s.batch * s.n_q_heads <= 5 * plan_cu_count();
}

// defer (with *deferred): when the one-pass kernel runs and the top-k that follows can take the merge
// of the output's partials into its own launch, that merge is not launched here but described in *defer.
static int focal_attn_score_impl(const fastocr_kv_view *kv, const fastocr_batch_view *bv, const void *q,
                                 int n_q_heads, float scale, void *out, float *scores, float *lse,
                                 float *img_mass, void *ws, size_t ws_bytes, void *hip_stream,
                                 const SelectArgs *select, bool *fused, CombineArgs *defer = nullptr, bool *deferred = nullptr)
{
    if (fused) *fused = false;
    if (deferred) *deferred = false;
    int rc = check_views(kv, bv, n_q_heads);
    if (rc != FASTOCR_OK) return rc;
    if (!out) return FASTOCR_EINVAL;
    rc = check_qo(kv, q, out, scale);
    if (rc != FASTOCR_OK) return rc;
    if (!scores && bv->max_vis_len > 0 && bv->batch > 0) return FASTOCR_EINVAL;
    const size_t need = fastocr_workspace_bytes(FASTOCR_OP_FOCAL_ATTN_SCORE, kv, bv, n_q_heads, 0);
    rc = check_ws(ws, ws_bytes, need);
    if (rc != FASTOCR_OK) return rc;
    if (bv->batch == 0) return FASTOCR_OK;
    Shape s = make_shape(kv, bv, n_q_heads);
    ResidentPlan rp;
    int slot = -1;
    uint32_t *flag = nullptr;
    // At head_dim 64 the layer has long been dense attention and then scoring: callers who overlap other work and keep its
    // scoring off the waiting grid ("score_resident" 0) have no such grid in this call either.
    const bool apart = kv->head_dim == 64 && g_tune_score_resident.load(std::memory_order_relaxed) == 0;
    const int mode = g_tune_focal_fused.load(std::memory_order_relaxed);
    const bool fuse = select && select_inside() && resident_select_fits(s);
    if (!apart && !parks(mode, s, kParkLayer) && use_resident(EX_FUSED, mode, s, &rp, (hipStream_t)hip_stream, &slot, &flag)) {
        const bool hand_on = defer && deferred && !fuse && merge_shares_topk(s);
        hipError_t e = launch_focal_fused(s, rp, slot, flag, q, scale, out, scores, lse, img_mass, ws, (hipStream_t)hip_stream,
                                          fuse ? select : nullptr, hand_on ? defer : nullptr);
        if (fused) *fused = fuse;
        if (hand_on) *deferred = true;
        return e == hipSuccess ? FASTOCR_OK : FASTOCR_EHIP;
    }
    if (parks_by_head(s) && !apart && mode != 0) {
        const bool hand_on = defer && deferred && !fuse && merge_shares_topk(s);
        const int nsplit = choose_splits(FASTOCR_OP_DENSE_DECODE_ATTN, s, bv->max_seq_len, nullptr, -1, true);
        const hipError_t e = launch_focal_parked(s, q, scale, out, scores, lse, img_mass, ws, nsplit, (hipStream_t)hip_stream,
                                                 fuse ? select : nullptr, hand_on ? defer : nullptr);
        if (fused) *fused = fuse;
        if (hand_on) *deferred = true;
        return e == hipSuccess ? FASTOCR_OK : FASTOCR_EHIP;
    }
    if (s.fast32 && mode != 0) {
        const bool hand_on = defer && deferred && merge_shares_topk(s);
        const int nsplit = choose_splits(FASTOCR_OP_DENSE_DECODE_ATTN, s, bv->max_seq_len);
        const hipError_t e = launch_focal_f32(s, q, scale, out, scores, lse, img_mass, ws, nsplit, (hipStream_t)hip_stream,
                                              hand_on ? defer : nullptr);
        if (hand_on) *deferred = true;
        return e == hipSuccess ? FASTOCR_OK : FASTOCR_EHIP;
    }
    rc = fastocr_dense_decode_attn(kv, bv, q, n_q_heads, scale, out, nullptr, ws, ws_bytes, hip_stream);
    if (rc != FASTOCR_OK) return rc;
    return focal_score_impl(kv, bv, q, n_q_heads, scale, scores, lse, img_mass, ws, ws_bytes, hip_stream, select, fused);
}

int fastocr_focal_attn_score(const fastocr_kv_view *kv, const fastocr_batch_view *bv, const void *q,
                             int n_q_heads, float scale, void *out, float *scores, float *lse,
                             float *img_mass, void *ws, size_t ws_bytes, void *hip_stream)
{
    return focal_attn_score_impl(kv, bv, q, n_q_heads, scale, out, scores, lse, img_mass, ws, ws_bytes, hip_stream, nullptr, nullptr);
}

int fastocr_focal_attn_score_topk(const fastocr_kv_view *kv, const fastocr_batch_view *bv, const void *q,
                                  int n_q_heads, float scale, double tau, const int32_t *prev_idx,
                                  const int32_t *prev_cnt, int32_t *sel_idx, int32_t *sel_cnt, int64_t kmax,
                                  void *out, float *scores, float *lse, float *img_mass, void *ws,
                                  size_t ws_bytes, void *hip_stream)
{
    int rc = check_topk_args(scores, bv, tau, prev_idx, prev_cnt, sel_idx, sel_cnt, kmax);
    if (rc != FASTOCR_OK) return rc;
    const size_t need = fastocr_workspace_bytes(FASTOCR_OP_FOCAL_ATTN_SCORE_TOPK, kv, bv, n_q_heads, kmax);
    if (need == 0) return check_views(kv, bv, n_q_heads) != FASTOCR_OK ? check_views(kv, bv, n_q_heads) : FASTOCR_EINVAL;
    rc = check_ws(ws, ws_bytes, need);
    if (rc != FASTOCR_OK) return rc;
    const SelectArgs sa{tau, prev_idx, prev_cnt, sel_idx, sel_cnt, kmax};
    bool fused = false, deferred = false;
    CombineArgs merge;
    rc = focal_attn_score_impl(kv, bv, q, n_q_heads, scale, out, scores, lse, img_mass, ws, ws_bytes, hip_stream, &sa, &fused,
                               &merge, &deferred);
    if (rc != FASTOCR_OK || fused) return rc;
    if (deferred) {
        // the merge of the output's partials and the top-k both wait for the one-pass kernel only: one launch
        // (the select keeps its keys in registers at these sizes and uses no workspace, the partials stay where they are)
        BatchDev bd{bv->seq_len, bv->vis_start, bv->vis_len, bv->max_seq_len, bv->max_vis_len};
        hipError_t e = launch_topk(scores, bd, bv->batch, tau, prev_idx, prev_cnt, sel_idx, sel_cnt, kmax, ws,
                                   (hipStream_t)hip_stream, &merge);
        return e == hipSuccess ? FASTOCR_OK : FASTOCR_EHIP;
    }
    return fastocr_topk_fixation(scores, bv, tau, prev_idx, prev_cnt, sel_idx, sel_cnt, kmax, ws, ws_bytes, hip_stream);
}

int fastocr_select_focal_layers(const float *ratio, int steps, int layers, int batch, double rho,
                                int gap, int32_t *focal_out, int32_t *n_out)
{
    if (!ratio || !focal_out || !n_out || steps < 1 || layers < 1 || batch < 1 || gap < 0) return FASTOCR_EINVAL;
    if (!(rho >= 0.0 && rho <= 1.0)) return FASTOCR_EINVAL;
    std::vector<double> mean((size_t)layers, 0.0);
    for (int t = 0; t < steps; ++t)
        for (int i = 0; i < layers; ++i)
            for (int b = 0; b < batch; ++b) {
                const float r = ratio[((size_t)t * layers + i) * batch + b];
                if (!isfinite(r)) return FASTOCR_EINVAL;
                mean[i] += (double)r;
            }
    for (int i = 0; i < layers; ++i) mean[i] /= (double)steps * (double)batch;
    std::vector<int> order((size_t)layers);
    for (int i = 0; i < layers; ++i) order[i] = i;
    std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return mean[x] > mean[y]; });
    const int budget = (int)floor(rho * (double)layers + 1e-9);
    std::vector<int> taken;
    for (int i : order) {
        if ((int)taken.size() >= budget) break;
        bool far = true;
        for (int j : taken) far = far && abs(i - j) > gap;
        if (far) taken.push_back(i);
    }
    std::sort(taken.begin(), taken.end());
    for (size_t x = 0; x < taken.size(); ++x) focal_out[x] = taken[x];
    *n_out = (int32_t)taken.size();
    return FASTOCR_OK;
}

int fastocr_kernel_timer_enable(int kernel, int capacity)
{
    if (kernel < 0 || kernel >= K_COUNT || capacity < 0) return FASTOCR_EINVAL;
    std::lock_guard<std::mutex> lock(g_mu);
    KernelTimer &t = g_timers[kernel];
    for (int i = 0; i < t.capacity; ++i) {
        (void)hipEventDestroy(t.start[i]);
        (void)hipEventDestroy(t.stop[i]);
    }
    delete[] t.start;
    delete[] t.stop;
    t = KernelTimer();
    if (capacity == 0) return FASTOCR_OK;
    t.start = new hipEvent_t[capacity];
    t.stop = new hipEvent_t[capacity];
    for (int i = 0; i < capacity; ++i) {
        if (hipEventCreate(&t.start[i]) != hipSuccess || hipEventCreate(&t.stop[i]) != hipSuccess) {
            t.capacity = 0;
            return FASTOCR_EHIP;
        }
    }
    t.capacity = capacity;
    return FASTOCR_OK;
}

int fastocr_kernel_timer_read(int kernel, float *ms_out, int max_out)
{
    if (kernel < 0 || kernel >= K_COUNT || (max_out > 0 && !ms_out)) return FASTOCR_EINVAL;
    std::lock_guard<std::mutex> lock(g_mu);
    KernelTimer &t = g_timers[kernel];
    const int n = t.count;
    for (int i = 0; i < n && i < max_out; ++i) {
        if (hipEventSynchronize(t.stop[i]) != hipSuccess) return FASTOCR_EHIP;
        if (hipEventElapsedTime(&ms_out[i], t.start[i], t.stop[i]) != hipSuccess) return FASTOCR_EHIP;
    }
    t.count = 0;
    return n;
}

int fastocr_stream_probe(const void *src, void *dst, size_t bytes, void *sink, void *hip_stream)
{
    if (!src || bytes < 16 || (reinterpret_cast<uintptr_t>(src) & 15u) || (reinterpret_cast<uintptr_t>(dst) & 15u))
        return FASTOCR_EINVAL;
    if (!dst && !sink) return FASTOCR_EINVAL;
    hipError_t e = launch_stream_probe(src, dst, bytes, sink, (hipStream_t)hip_stream);
    return e == hipSuccess ? FASTOCR_OK : FASTOCR_EHIP;
}

int fastocr_stream_release(void *hip_stream)
{
    // the slot numbers of the streams that stay must not move (their calls may be in flight), so a
    // released entry is only marked free and handed to the next stream that asks
    std::lock_guard<std::mutex> lock(g_mu);
    for (int kind = 0; kind < EX_KINDS; ++kind)
        for (int dev = 0; dev < kMaxDevices; ++dev)
            for (SlotOwner &o : g_slots[kind][dev].eager)
                if (!o.free && o.stream == (hipStream_t)hip_stream) o.free = true;
    return FASTOCR_OK;
}

int fastocr_exchange_timeouts(uint64_t *count)
{
    if (!count) return FASTOCR_EINVAL;
    uint32_t a = 0, b = 0, c = 0;
    if (score_resident_timeouts(&a) != hipSuccess || focal_fused_timeouts(&b) != hipSuccess ||
        attn_merge_timeouts(&c) != hipSuccess)
        return FASTOCR_EHIP;
    *count = (uint64_t)a + b + c;
    return FASTOCR_OK;
}

int fastocr_set_tuning(const char *key, int value)
{
    if (!key || value < 0) return FASTOCR_EINVAL;
    if (!strcmp(key, "splits_score")) g_tune_splits[FASTOCR_OP_FOCAL_SCORE] = value;
    else if (!strcmp(key, "splits_sparse")) g_tune_splits[FASTOCR_OP_SPARSE_DECODE_ATTN] = value;
    else if (!strcmp(key, "splits_dense")) g_tune_splits[FASTOCR_OP_DENSE_DECODE_ATTN] = value;
    else if (!strcmp(key, "attn_waves") && (value == 4 || value == 8)) g_tune_attn_waves = value;
    else if (!strcmp(key, "graph_replay") && (value == 0 || value == 1)) g_tune_graph_replay = value;
    else if (!strcmp(key, "timer_every") && value >= 1) g_tune_timer_every = value;
    else if (!strcmp(key, "attn_merge") && value <= 2) g_tune_attn_merge = value;
    else if (!strcmp(key, "barrier_spin_us")) g_tune_barrier_spin_us = value ? value : 250000;
    else if (!strcmp(key, "score_resident") && value <= 2) g_tune_score_resident = value;
    else if (!strcmp(key, "focal_fused") && value <= 2) g_tune_focal_fused = value;
    else if (!strcmp(key, "select_fused") && value <= 1) g_tune_select_fused = value;
    else if (!strcmp(key, "exchange_fallback") && value <= 1) {
        g_exchange_distrusted = value;
        if (value == 0) {
            // re-arm: forget that waves have given up (the caller has taken the other work off the GPU)
            std::lock_guard<std::mutex> lock(g_mu);
            for (int d = 0; d < kMaxDevices; ++d)
                if (g_gave_up[d]) __atomic_store_n(g_gave_up[d], 0u, __ATOMIC_RELAXED);
        }
    }
    else return FASTOCR_EINVAL;
    return FASTOCR_OK;
}

const char *fastocr_strerror(int status)
{
    switch (status) {
    case FASTOCR_OK: return "ok";
    case FASTOCR_EINVAL: return "invalid argument";
    case FASTOCR_EUNSUPPORTED: return "unsupported dtype, head_dim or head count";
    case FASTOCR_EWORKSPACE: return "workspace missing, misaligned or too small";
    case FASTOCR_EHIP: return "HIP runtime error";
    case FASTOCR_ETOOLARGE: return "shape needs more scratch than the library's static buffer holds (FASTOCR_STATIC_SCRATCH_BYTES)";
    default: return "unknown status";
    }
}

const char *fastocr_version(void) { return "fastocr-mi355x 0.1 (gfx950)"; }

}  // extern "C"
