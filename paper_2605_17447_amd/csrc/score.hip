// Focal-layer scoring: head-averaged softmax attention of the current query over the whole
// cache, read at the image tokens (Eq. 1; text under Eq. 2).
//
// The average over heads is taken AFTER each head's softmax, so no score is final before
// every head's normaliser over all S keys is known.  Two launches:
//   logits : streams K once (for a focal layer K and V).  Per (sequence, kv head, token range) it computes the query heads' logits, parks
//            them (fp32, log2 domain) in the workspace and leaves a per-range (max, sum-exp) per head.  bf16 caches of head_dim 128 and
//            64: attn.hip (kLogits, kParked); fp32 caches of these: attn_f32.hip; otherwise the plain kernel here.
//   finish : merges the per-range statistics into each head's maximum M and sum Z and writes
//            score_i = (1/Hq) sum_h 2^(logit_h,i - M_h) / Z_h for the image tokens; for bf16 also the image mass and the merge of
//            the output's partials.
#include "kernels.hpp"
#include "combine.hpp"
#include "topk_dev.hpp"

namespace fastocr {

// Parked logits, fp32.  bf16 on the matrix cores (attn.hip, kLogits and kParked): [sequence][query head][token (pitch)].  Otherwise
// [sequence][kv head][token (pitch)][Gp], Gp = G rounded up to 4 heads.
__host__ __device__ inline int park_heads(int G) { return (G + 3) / 4 * 4; }

// Generic (fp32 caches of head_dim 128 and 64 take attn_f32.hip): one wave per (range, query head, sequence), lanes over tokens.  The q.k sums run in
// fp64 (dot_row) and are scaled there; the logit is rounded to fp32 once, when it is parked.
template <typename T, bool PAGED>
__global__ __launch_bounds__(64) void score_generic_kernel(
    KvDev kv, BatchDev bv, const T *__restrict__ q, int Hq, double scale_log2,
    float *__restrict__ logits, int64_t pitch, float *__restrict__ part_ml, int nsplit, bool vec16)
{
    __shared__ float qs[256];
    const int lane = threadIdx.x;
    const int split = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
    const int d = kv.head_dim;
    const int G = Hq / kv.n_kv_heads, Gp = park_heads(G);
    const int g = h / G;
    const SeqGeom geo = seq_geom(bv, b);
    const int L = geo.S;
    const int ntile = (L + 63) / 64;
    const int tps = (ntile + nsplit - 1) / nsplit;
    const int t0 = split * tps, t1 = min(ntile, t0 + tps);

    for (int c = lane; c < d; c += 64) qs[c] = load_elem<T>(q + ((int64_t)b * Hq + h) * d + c);
    __syncthreads();
    const T *kbase = reinterpret_cast<const T *>(kv.k);
    float *lrow = logits + ((int64_t)b * kv.n_kv_heads + g) * pitch * Gp + (h - g * G);   // [token][Gp]
    float m = kMinusHuge, z = 0.f;
    for (int tile = t0; tile < t1; ++tile) {
        const int p = tile * 64 + lane;
        const bool valid = p < L;
        const int64_t off = row_offset<PAGED>(kv, b, min(p, L - 1), g);
        const float s = valid ? (float)(dot_row<T>(qs, kbase + off, d, vec16) * scale_log2) : -INFINITY;
        lrow[(int64_t)p * Gp] = s;                       // p < pitch: pitch is a multiple of 64
        const float m_new = fmaxf(m, wave_max(s));
        z = z * fast_exp2(m - m_new) + wave_sum(fast_exp2(s - m_new));
        m = m_new;
    }
    if (lane == 0) {
        const int64_t ph = ((int64_t)b * Hq + h) * nsplit + split;
        part_ml[ph * 2] = m;
        part_ml[ph * 2 + 1] = z;
    }
}

// Finalize: per-head log-sum-exp from the range statistics, then the head average
//     score_i = (1/Hq) sum_h 2^(logit_h,i - lse_h)
// read back from the parked [token][Gp] rows.  LP lanes share a token (one 16-byte quad of heads
// per kv head each), so that a wave's loads cover contiguous memory.
constexpr int kFinThreads = 256;

__host__ __device__ inline int fin_lanes_per_token(int Gp) { return Gp == 8 ? 2 : (Gp == 16 ? 4 : 1); }

__global__ __launch_bounds__(kFinThreads) void score_finalize_kernel(
    const float *__restrict__ part_ml, const float *__restrict__ logits, const int32_t *__restrict__ seq_len,
    const int32_t *__restrict__ vis_start, const int32_t *__restrict__ vis_len, int64_t pitch, int Hq, int nsplit,
    int n_kv_heads, int max_seq_len, int max_vis_len, float *__restrict__ scores, float *__restrict__ lse, float *__restrict__ mass_part)
{
    const BatchDev bv{seq_len, vis_start, vis_len, max_seq_len, max_vis_len};
    // [Hq][2]: a head's maximum M and 1/Z over the sequence.  A weight is 2^(logit - M) / Z: the difference of two
    // logits of like size is nearly exact, where logit - (M + log2 Z) would carry the rounding of that sum
    extern __shared__ float norm[];
    __shared__ float red[kFinThreads / 64];
    const int b = blockIdx.y;
    const SeqGeom geo = seq_geom(bv, b);
    // every head's log-sum-exp from its nsplit range statistics: 8 lanes share a head and walk every
    // 8th range (a serial walk is bound by load latency once there are dozens of ranges)
    for (int h0 = 0; h0 < Hq; h0 += kFinThreads / 8) {
        const int h = h0 + (threadIdx.x >> 3), part = threadIdx.x & 7;
        float M = kMinusHuge, Z = 0.f;
        if (h < Hq) {
            const float *ml = part_ml + ((int64_t)b * Hq + h) * nsplit * 2;
            for (int s = part; s < nsplit; s += 8) softmax_merge(M, Z, ml[2 * s], ml[2 * s + 1]);
        }
#pragma unroll
        for (int o = 1; o < 8; o <<= 1) softmax_merge(M, Z, __shfl_xor(M, o), __shfl_xor(Z, o));
        if (h < Hq && part == 0) {
            norm[2 * h] = M;
            norm[2 * h + 1] = 1.0f / Z;
            if (lse && blockIdx.x == 0) lse[(int64_t)b * Hq + h] = (Z > 0.f ? M + log2f(Z) : -INFINITY) * kLn2;
        }
    }
    __syncthreads();
    const int G = Hq / n_kv_heads, Gp = park_heads(G);
    const int LP = fin_lanes_per_token(Gp);
    const int nq = Gp / 4 / LP;                        // 16-byte quads per lane per kv head
    const int i = (blockIdx.x * kFinThreads + threadIdx.x) / LP;
    const int sub = threadIdx.x % LP;
    float acc = 0.f;
    if (i < geo.N) {
        const float *lp = logits + ((int64_t)b * n_kv_heads * pitch + geo.v0 + i) * Gp;
        for (int g = 0; g < n_kv_heads; ++g) {
            const float *row = lp + (int64_t)g * pitch * Gp;
            for (int qd = 0; qd < nq; ++qd) {
                const int x0 = 4 * (sub * nq + qd);
                const f32x4 v = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(row + x0));
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (x0 + r < G) acc += fast_exp2(v[r] - norm[2 * (g * G + x0 + r)]) * norm[2 * (g * G + x0 + r) + 1];
            }
        }
    }
    for (int o = 1; o < LP; o <<= 1) acc += __shfl_xor(acc, o);
    float sc = 0.f;
    if (i < geo.N && sub == 0) {
        sc = acc / (float)Hq;
        scores[(int64_t)b * bv.max_vis_len + i] = sc;
    }
    if (mass_part) {
        float w = wave_sum(sc);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = w;
        __syncthreads();
        if (threadIdx.x == 0) {
            float t = 0.f;
            for (int x = 0; x < kFinThreads / 64; ++x) t += red[x];
            mass_part[(int64_t)b * gridDim.x + blockIdx.x] = t;
        }
    }
}

__global__ void mass_reduce_kernel(const float *__restrict__ mass_part, int nblk, float *__restrict__ img_mass)
{
    const int b = blockIdx.x;
    float t = 0.f;
    for (int x = threadIdx.x; x < nblk; x += 64) t += mass_part[(int64_t)b * nblk + x];
    t = wave_sum(t);
    if (threadIdx.x == 0) img_mass[b] = t;
}


// ---- bf16: what follows the kernels that park logits as [sequence][query head][token] ------------------------------------
// One launch of up to three kinds of workgroup, none of which waits for another: the scores of 64 tokens each, the image mass of
// a sequence, the merge of one query head's output partials.  Bound by latency (a few MB): every load a workgroup of the
// first kind needs -- its logits and its heads' statistics, whose addresses do not depend on the sequence's geometry -- is
// requested at once, one memory round trip; 16 lanes share a head and merge its ranges with lane moves, the heads of a token meet
// by half swaps and one trip through LDS.
constexpr int kFinTokens = 64;

// (M, Z) of NU heads hg, hg + 16, .. over their nsplit ranges, and the image tokens' part of Z with MASS, in all 16 lanes of a row.
// NS: ranges per lane requested at a time, 16 NS in all (1: up to 16 ranges in one round trip, 4: up to 64).  meanwhile(): what is
// done while they are on their way.
template <int NU, int NS, bool MASS, typename F>
__device__ __forceinline__ void parked_stats(const float *__restrict__ part_ml, const float *__restrict__ part_zi, int64_t bh0, int h0, int Hq,
                                             int nsplit, float (&M)[NU], float (&Z)[NU], float (&Zi)[NU], F meanwhile)
{
    const int tq = threadIdx.x & 15;
#pragma unroll
    for (int u = 0; u < NU; ++u) { M[u] = kLowest; Z[u] = 0.f; Zi[u] = 0.f; }
    for (int s0 = 0; s0 < nsplit; s0 += 16 * NS) {
        float mm[NU][NS], zz[NU][NS], ii[NU][NS];
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int64_t row = (bh0 + min(h0 + 16 * u, Hq - 1)) * nsplit;
#pragma unroll
            for (int k = 0; k < NS; ++k) {
                const int s = s0 + 16 * k + tq;
                const int64_t at = row + min(s, nsplit - 1);
                const float2 ml = *reinterpret_cast<const float2 *>(part_ml + 2 * at);
                mm[u][k] = s < nsplit ? ml.x : kLowest;
                zz[u][k] = s < nsplit ? ml.y : 0.f;
                ii[u][k] = MASS ? (s < nsplit ? part_zi[at] : 0.f) : 0.f;
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        meanwhile();
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            float mx = M[u];
#pragma unroll
            for (int k = 0; k < NS; ++k) mx = fmaxf(mx, mm[u][k]);
            const float f0 = fast_exp2(M[u] - mx);
            Z[u] *= f0;
            if (MASS) Zi[u] *= f0;
#pragma unroll
            for (int k = 0; k < NS; ++k) {
                const float f = fast_exp2(mm[u][k] - mx);
                Z[u] += zz[u][k] * f;
                if (MASS) Zi[u] += ii[u][k] * f;
            }
            M[u] = mx;
        }
    }
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        float mx = M[u];
        mx = fmaxf(mx, dpp_move<kDppXor1>(mx));
        mx = fmaxf(mx, dpp_move<kDppXor2>(mx));
        mx = fmaxf(mx, dpp_move<kDppHalfMirror>(mx));
        mx = fmaxf(mx, dpp_move<kDppRowMirror>(mx));
        const float f = fast_exp2(M[u] - mx);
        float z = Z[u] * f, zi = MASS ? Zi[u] * f : 0.f;
        z += dpp_move<kDppXor1>(z);
        z += dpp_move<kDppXor2>(z);
        z += dpp_move<kDppHalfMirror>(z);
        z += dpp_move<kDppRowMirror>(z);
        if (MASS) {
            zi += dpp_move<kDppXor1>(zi);
            zi += dpp_move<kDppXor2>(zi);
            zi += dpp_move<kDppHalfMirror>(zi);
            zi += dpp_move<kDppRowMirror>(zi);
        }
        M[u] = mx;
        Z[u] = z;
        Zi[u] = zi;
    }
}

// Scores of the 64 tokens of block `blk` by 256 consecutive threads (all threads of the workgroup call: a barrier inside).
// NU: sixteenths of the query heads a lane looks after at a time (1, 2, 4: up to 16, 32, 64 heads; more heads in rounds).
// COHERENT: stored for a reader in the same launch.
template <int NU, int NS, bool COHERENT>
__device__ __forceinline__ void parked_scores(const BatchDev &bv, int b, int blk, int Hq, const float *__restrict__ logits, int64_t pitch,
                                              const float *__restrict__ part_ml, int nsplit, float *__restrict__ scores,
                                              float *__restrict__ lse, float *sm)
{
    const int t = threadIdx.x & 255, tq = t & 15, hg = t >> 4, wave = t >> 6;
    const int64_t bh0 = (int64_t)b * Hq;
    const int p0 = blk * kFinTokens + 4 * tq;                    // tokens of the sequence
    const int at = parked_token(p0, pitch);
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
    // The geometry is read through the scalar cache while logits and statistics come.  (Named where it is used, behind the sums, the compiler asks for
    // it there: one more round trip before the store.)
    int s_len = 0, v_start = 0, v_len = 0;
    auto geometry = [&]() {
        s_len = bv.seq_len[b];
        v_start = bv.vis_start[b];
        v_len = bv.vis_len[b];
        asm volatile("" : "+s"(s_len), "+s"(v_start), "+s"(v_len));
    };
    for (int r0 = 0; r0 < Hq; r0 += 16 * NU) {                   // (every lane walks every round)
        const int h0 = r0 + hg;
        f32x4 l[NU];
#pragma unroll
        for (int u = 0; u < NU; ++u)
            l[u] = *reinterpret_cast<const f32x4 *>(logits + (bh0 + min(h0 + 16 * u, Hq - 1)) * pitch + at);
        float M[NU], Z[NU], unused[NU];
        parked_stats<NU, NS, false>(part_ml, nullptr, bh0, h0, Hq, nsplit, M, Z, unused, geometry);
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const bool there = h0 + 16 * u < Hq;
            const float inv = 1.0f / Z[u];
            // relative to the head's maximum: the difference of two logits of like size is nearly exact
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] += there ? fast_exp2(l[u][e] - M[u]) * inv : 0.f;
            if (lse && blk == 0 && tq == 0 && there) lse[bh0 + h0 + 16 * u] = (Z[u] > 0.f ? M[u] + log2f(Z[u]) : -INFINITY) * kLn2;
        }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] = rows_sum(acc[e]);       // the wave's four head groups
    if ((t & 63) < 16) *reinterpret_cast<f32x4 *>(&sm[wave * kFinTokens + 4 * tq]) = acc;
    const SeqGeom geo = seq_geom_of(bv, s_len, v_start, v_len);
    __syncthreads();
    if (t < kFinTokens) {
        const int i = blk * kFinTokens + t - geo.v0;
        const float sum = (sm[t] + sm[kFinTokens + t]) + (sm[2 * kFinTokens + t] + sm[3 * kFinTokens + t]);
        if (i >= 0 && i < geo.N) {
            float *to = &scores[(int64_t)b * bv.max_vis_len + i];
            if (COHERENT) __hip_atomic_store(to, sum / (float)Hq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            else *to = sum / (float)Hq;
        }
    }
}

// Image mass of sequence b by 256 threads of a workgroup all of which call: the sum of its scores, no number where they are none.
template <int NU, int NS>
__device__ __forceinline__ void parked_mass(const BatchDev &bv, int b, int Hq, const float *__restrict__ part_ml, const float *__restrict__ part_zi, int nsplit,
                                            float *__restrict__ img_mass, float *sm)
{
    const int t = threadIdx.x & 255, hg = t >> 4;
    float sum = 0.f;
    for (int h0 = hg; h0 < Hq + hg; h0 += 16 * NU) {
        float M[NU], Z[NU], Zi[NU];
        parked_stats<NU, NS, true>(part_ml, part_zi, (int64_t)b * Hq, h0, Hq, nsplit, M, Z, Zi, []() {});
#pragma unroll
        for (int u = 0; u < NU; ++u) sum += h0 + 16 * u < Hq ? Zi[u] / Z[u] : 0.f;
    }
    sum = rows_sum(sum);
    if (threadIdx.x < 256 && (t & 63) == 0) sm[t >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) img_mass[b] = seq_geom(bv, b).N > 0 ? ((sm[0] + sm[1]) + (sm[2] + sm[3])) / (float)Hq : 0.f;
}

template <int NU, int NS>
__global__ __launch_bounds__(kFinThreads) void parked_finish_kernel(
    const float *__restrict__ logits, const float *__restrict__ part_ml, const float *__restrict__ part_o, const float *__restrict__ part_zi,
    int64_t pitch, int Hq, int nsplit, int nblk, int d, const int32_t *__restrict__ seq_len, const int32_t *__restrict__ vis_start,
    const int32_t *__restrict__ vis_len, int max_seq_len, int max_vis_len, float *__restrict__ scores, float *__restrict__ lse,
    float *__restrict__ img_mass, uint16_t *__restrict__ out)
{
    const BatchDev bv{seq_len, vis_start, vis_len, max_seq_len, max_vis_len};
    __shared__ float sm_max[4];
    __shared__ float sm_z[256];
    __shared__ __align__(16) float sm_o[1024];
    const int b = blockIdx.y, blk = blockIdx.x;
    if (blk < nblk) parked_scores<NU, NS, false>(bv, b, blk, Hq, logits, pitch, part_ml, nsplit, scores, lse, sm_o);
    else if (img_mass && blk == nblk) parked_mass<NU, NS>(bv, b, Hq, part_ml, part_zi, nsplit, img_mass, sm_max);
    else combine_wide_body<uint16_t>(part_o, part_ml, nsplit, d, out, nullptr, nullptr, 1, blk - nblk - (img_mass ? 1 : 0), b, Hq,
                                     CombineShared<uint16_t>{sm_max, sm_z, sm_o});
}

// The same with the top-k of the scores in the launch ("select_fused" 1): workgroups of 1024 threads, 256 tokens each, count themselves out per
// sequence (`done`, zeroed by the launch before) once their scores, stored at agent scope, have been performed; the
// sequence's last one selects over all of them as topk_reg_kernel does, with the same bits.  Nobody waits for anybody.  Not the
// default: the count and the scores' way back through memory cost more than a launch (a layer with its top-k, separate launches /
// this one, us: 28/4 heads, batch 1, 4096 image tokens 14.8 / 16.1, 16384 22.0 / 28.7, 12 x 4096 31.3 / 33.4).
constexpr int kFinSelThreads = 1024;
constexpr int kFinSelBlocks = kFinSelThreads / 256;          // 64-token blocks per workgroup

__global__ __launch_bounds__(kFinSelThreads) void parked_select_kernel(
    const int32_t *__restrict__ seq_len, const int32_t *__restrict__ vis_start, const int32_t *__restrict__ vis_len, int max_seq_len, int max_vis_len,
    int Hq, const float *__restrict__ logits, int64_t pitch, const float *__restrict__ part_ml,
    const float *__restrict__ part_zi, int nsplit, float *__restrict__ scores, float *__restrict__ lse, float *__restrict__ img_mass,
    int nwg, const float *__restrict__ part_o, int d, uint16_t *__restrict__ out, SelectArgs sel, uint32_t *__restrict__ done)
{
    const BatchDev bv{seq_len, vis_start, vis_len, max_seq_len, max_vis_len};
    __shared__ uint32_t hist[kWinBins];
    __shared__ __align__(16) uint32_t list[kWinListWords];
    __shared__ int s_pick[4];
    __shared__ __align__(16) int w_ac[6 * (kFinSelThreads / 64)];
    __shared__ float sm_max[4];
    __shared__ float sm_z[256];
    __shared__ __align__(16) float sm_o[1024];
    __shared__ int s_last;
    const int b = blockIdx.y, wg = blockIdx.x;
    if (wg >= nwg) {
        if (img_mass && wg == nwg) parked_mass<4, 4>(bv, b, Hq, part_ml, part_zi, nsplit, img_mass, sm_max);
        else combine_wide_body<uint16_t>(part_o, part_ml, nsplit, d, out, nullptr, nullptr, 1, wg - nwg - (img_mass ? 1 : 0), b, Hq,
                                         CombineShared<uint16_t>{sm_max, sm_z, sm_o});
        return;
    }
    const int sub = threadIdx.x >> 8;
    parked_scores<4, 4, true>(bv, b, wg * kFinSelBlocks + sub, Hq, logits, pitch, part_ml, nsplit, scores, lse, sm_o + 256 * sub);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // this thread's scores have been performed
    __syncthreads();                                         // ... and every other thread's of the workgroup
    if (threadIdx.x == 0)
        s_last = __hip_atomic_fetch_add(&done[b], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)nwg - 1u;
    __syncthreads();
    if (!s_last) return;
    TopkRegShared sh;
    sh.hist = hist; sh.list = list; sh.pick = s_pick; sh.w_ac = w_ac;
    topk_reg_body<kFinSelThreads, 16, true, false>(scores, bv, b, sel.tau, sel.prev_idx, sel.prev_cnt, sel.sel_idx, sel.sel_cnt, sel.kmax, sh);
}

// -----------------------------------------------------------------------------------------
static int fin_blocks(const Shape &s)
{
    const int LP = fin_lanes_per_token(park_heads(s.n_q_heads / s.kv.n_kv_heads));
    const int per = kFinThreads / LP;
    return max(1, (s.bv.max_vis_len + per - 1) / per);
}

bool parks_by_head(const Shape &s)
{
    // a group's rows are addressed with 32-bit byte offsets
    return mfma_path(s) && (s.n_q_heads / s.kv.n_kv_heads) * logit_pitch(s.bv.max_seq_len) < ((int64_t)1 << 29);
}

static size_t parked_floats(const Shape &s)
{
    const size_t pitch = (size_t)logit_pitch(s.bv.max_seq_len);
    if (parks_by_head(s)) return (size_t)s.batch * s.n_q_heads * pitch;
    return (size_t)s.batch * s.kv.n_kv_heads * pitch * park_heads(s.n_q_heads / s.kv.n_kv_heads);
}

size_t score_workspace_bytes(const Shape &s, size_t rows)
{
    size_t bytes = parked_floats(s) * sizeof(float);
    bytes += rows * (parks_by_head(s) ? 3 : 2) * sizeof(float);
    if (parks_by_head(s)) bytes += (size_t)s.batch * sizeof(uint32_t);
    if (!parks_by_head(s)) bytes += (size_t)s.batch * fin_blocks(s) * sizeof(float);
    return bytes;
}

static hipError_t launch_finalize(const Shape &s, const float *logits, int64_t pitch, const float *part_ml, int nsplit,
                                  float *scores, float *lse, float *img_mass, float *mass_part, hipStream_t stream)
{
    const int nblk = fin_blocks(s);
    dim3 fgrid(nblk, s.batch), fblock(kFinThreads);
    FASTOCR_LAUNCH(K_SCORE_FINALIZE, score_finalize_kernel, fgrid, fblock, (size_t)s.n_q_heads * 2 * sizeof(float), stream,
        part_ml, logits, s.bv.seq_len, s.bv.vis_start, s.bv.vis_len, pitch, s.n_q_heads, nsplit, s.kv.n_kv_heads, s.bv.max_seq_len, s.bv.max_vis_len,
        scores, lse, img_mass ? mass_part : nullptr);
    return hipGetLastError();
}

// part_o, out: the merge of the output's partials as well (null: scores alone).  select: the top-k as well (parked_select_fits).
static hipError_t launch_parked_finish(const Shape &s, const float *logits, int64_t pitch, const float *part_ml, const float *part_zi, int nsplit,
                                       float *scores, float *lse, float *img_mass, const float *part_o, void *out,
                                       const SelectArgs *select, uint32_t *done, hipStream_t stream)
{
    if (select) {
        const int nwg = std::max(1, (s.bv.max_seq_len + kFinSelBlocks * kFinTokens - 1) / (kFinSelBlocks * kFinTokens));
        const dim3 grid(nwg + (img_mass ? 1 : 0) + (out ? s.n_q_heads : 0), s.batch), block(kFinSelThreads);
        FASTOCR_LAUNCH(K_PARKED_FINISH, parked_select_kernel, grid, block, 0, stream, s.bv.seq_len, s.bv.vis_start, s.bv.vis_len, s.bv.max_seq_len, s.bv.max_vis_len, s.n_q_heads, logits, pitch, part_ml, part_zi, nsplit, scores, lse,
                       img_mass, nwg, part_o, s.kv.head_dim, (uint16_t *)out, *select, done);
        return hipGetLastError();
    }
    // Over the longest sequence's tokens, so that no load waits for where an image starts or a sequence ends: workgroups without image tokens read
    // words that nobody wrote and drop what they make of them.
    const int nblk = std::max(1, (s.bv.max_seq_len + kFinTokens - 1) / kFinTokens);
    const dim3 grid(nblk + (img_mass ? 1 : 0) + (out ? s.n_q_heads : 0), s.batch), block(kFinThreads);
#define FASTOCR_FINISH_N(NU, NS) FASTOCR_LAUNCH(K_PARKED_FINISH, (parked_finish_kernel<NU, NS>), grid, block, 0, stream, logits, part_ml, part_o, part_zi, \
        pitch, s.n_q_heads, nsplit, nblk, s.kv.head_dim, s.bv.seq_len, s.bv.vis_start, s.bv.vis_len, s.bv.max_seq_len, s.bv.max_vis_len, scores, lse, img_mass, (uint16_t *)out)
#define FASTOCR_FINISH(NU) do { if (nsplit <= 16) FASTOCR_FINISH_N(NU, 1); else FASTOCR_FINISH_N(NU, 4); } while (0)
    if (s.n_q_heads <= 16) FASTOCR_FINISH(1);
    else if (s.n_q_heads <= 32) FASTOCR_FINISH(2);
    else FASTOCR_FINISH(4);
#undef FASTOCR_FINISH
#undef FASTOCR_FINISH_N
    return hipGetLastError();
}

hipError_t launch_score(const Shape &s, const void *q, float scale, float *scores, float *lse,
                        float *img_mass, void *ws, int nsplit, hipStream_t stream, const SelectArgs *select)
{
    const int64_t pitch = logit_pitch(s.bv.max_seq_len);
    const size_t rows = (size_t)s.batch * s.n_q_heads;
    float *logits = reinterpret_cast<float *>(ws);
    float *part_ml = logits + parked_floats(s);
    if (parks_by_head(s)) {
        float *part_zi = img_mass ? part_ml + rows * nsplit * 2 : nullptr;
        uint32_t *done = select ? reinterpret_cast<uint32_t *>(part_ml + rows * nsplit * 3) : nullptr;
        const hipError_t e = launch_attn_parked(K_SCORE_LOGITS, s, q, scale, nullptr, part_ml, part_zi, nsplit, logits, pitch, done, stream);
        if (e != hipSuccess) return e;
        return launch_parked_finish(s, logits, pitch, part_ml, part_zi, nsplit, scores, lse, img_mass, nullptr, nullptr,
                                    select, done, stream);
    }
    float *mass_part = part_ml + rows * nsplit * 2;
    const int G = s.n_q_heads / s.kv.n_kv_heads;
    if (f32_mfma_path(s)) {
        const hipError_t e = launch_attn_f32(K_SCORE_LOGITS, s, q, scale, nullptr, nullptr, 0, nullptr, part_ml, nsplit, nullptr, nullptr,
                                             logits, pitch, stream);
        if (e != hipSuccess) return e;
    } else {
        dim3 grid(nsplit, s.n_q_heads, s.batch), block(64);
#define FASTOCR_SCORE(T, P) FASTOCR_LAUNCH(K_SCORE_LOGITS, (score_generic_kernel<T, P>), grid, block, 0, stream, \
        s.kv, s.bv, (const T *)q, s.n_q_heads, (double)scale * 1.4426950408889634074, logits, pitch, part_ml, nsplit, s.vec16)
        if (s.dtype == DT_BF16) { if (s.paged) FASTOCR_SCORE(uint16_t, true); else FASTOCR_SCORE(uint16_t, false); }
        else                    { if (s.paged) FASTOCR_SCORE(float, true); else FASTOCR_SCORE(float, false); }
#undef FASTOCR_SCORE
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;

    e = launch_finalize(s, logits, pitch, part_ml, nsplit, scores, lse, img_mass, mass_part, stream);
    if (e != hipSuccess || !img_mass) return e;
    mass_reduce_kernel<<<s.batch, 64, 0, stream>>>(mass_part, fin_blocks(s), img_mass);
    return hipGetLastError();
}

// A focal layer of a bf16 cache as two launches: attention partials and parked logits, then scores, image mass and (unless it is
// handed on to the top-k's launch) the output's merge at once.
// Workspace: logits, the attention partials fp32 [rows][d], the ranges' statistics [rows][2] and image sums [rows], a count per sequence.
size_t focal_parked_workspace_bytes(const Shape &s, size_t rows)
{
    return (parked_floats(s) + rows * (3 + s.kv.head_dim) + s.batch) * sizeof(float);
}

hipError_t launch_focal_parked(const Shape &s, const void *q, float scale, void *out, float *scores, float *lse, float *img_mass,
                               void *ws, int nsplit, hipStream_t stream, const SelectArgs *select, CombineArgs *defer)
{
    const int64_t pitch = logit_pitch(s.bv.max_seq_len);
    const size_t rows = (size_t)s.batch * s.n_q_heads * nsplit;
    float *logits = reinterpret_cast<float *>(ws);
    float *part_o = logits + parked_floats(s);                       // 16-byte aligned: the pitch is a multiple of 64
    float *part_ml = part_o + rows * s.kv.head_dim;
    float *part_zi = img_mass ? part_ml + rows * 2 : nullptr;
    uint32_t *done = select ? reinterpret_cast<uint32_t *>(part_ml + rows * 3) : nullptr;
    const hipError_t e = launch_attn_parked(K_FOCAL_FUSED, s, q, scale, part_o, part_ml, part_zi, nsplit, logits, pitch, done, stream);
    if (e != hipSuccess) return e;
    const bool hand_on = defer && !select;
    if (hand_on) *defer = CombineArgs{part_o, part_ml, nsplit, s.kv.head_dim, s.n_q_heads, 1, nullptr, out, false, MassArgs{nullptr, nullptr, 0}};
    return launch_parked_finish(s, logits, pitch, part_ml, part_zi, nsplit, scores, lse, img_mass,
                                hand_on ? nullptr : part_o, hand_on ? nullptr : out, select, done, stream);
}

// Workspace: as launch_score's, then the attention partials fp32 [B][Hq][nsplit][d] (the softmax statistics serve both).
size_t focal_f32_workspace_bytes(const Shape &s, size_t rows)
{
    return (score_workspace_bytes(s, rows) + 255) / 256 * 256 + rows * s.kv.head_dim * sizeof(float);
}

hipError_t launch_focal_f32(const Shape &s, const void *q, float scale, void *out, float *scores, float *lse, float *img_mass,
                            void *ws, int nsplit, hipStream_t stream, CombineArgs *defer)
{
    const int64_t pitch = logit_pitch(s.bv.max_seq_len);
    float *logits = reinterpret_cast<float *>(ws);
    float *part_ml = logits + parked_floats(s);
    const size_t rows = (size_t)s.batch * s.n_q_heads * nsplit;
    float *mass_part = part_ml + rows * 2;
    float *part_o = logits + (score_workspace_bytes(s, rows) + 255) / 256 * 256 / sizeof(float);
    hipError_t e = launch_attn_f32(K_FOCAL_FUSED, s, q, scale, nullptr, nullptr, 0, part_o, part_ml, nsplit, nullptr, nullptr, logits,
                                   pitch, stream);
    if (e != hipSuccess) return e;
    e = launch_finalize(s, logits, pitch, part_ml, nsplit, scores, lse, img_mass, mass_part, stream);
    if (e != hipSuccess) return e;
    const MassArgs mass{mass_part, img_mass, fin_blocks(s)};
    if (defer) {
        *defer = CombineArgs{part_o, part_ml, nsplit, s.kv.head_dim, s.n_q_heads, 1, nullptr, out, true, mass};
        return hipSuccess;
    }
    return launch_attn_combine(s, part_o, part_ml, nsplit, out, nullptr, stream, nullptr, 1, mass);
}

}  // namespace fastocr
