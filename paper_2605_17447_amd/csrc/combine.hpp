// Merge of attention partials spread over a workgroup's threads, as a device function: the merge kernel
// of attn.hip is this body, and so are the extra workgroups of the launch that runs a focal layer's
// top-k (topk.hip) -- the two depend only on the one-pass kernel before them, so they share a launch.
#pragma once
#include "kernels.hpp"

namespace fastocr {

constexpr int kCombineWalk = 12;       // up to this many every thread walks their maxima
constexpr int kCombineFew = 32;        // up to this many partials per head the merge takes its one-round-trip form

// What the partials are added up in: fp64 for fp32 outputs (up to 32 and more fp32 partials in an fp32 chain were the
// largest part of those outputs' error), else fp32.
template <typename T> struct CombineAcc { typedef float type; };
template <> struct CombineAcc<float> { typedef double type; };

template <typename T>
struct CombineShared {
    typedef typename CombineAcc<T>::type A;
    float *max4;        // [4]
    A *z;               // [256]
    A *o;               // [1024], 16-byte aligned: [split lane][d], SL * d <= 1024 as DL >= d/4
};

// out = sum_s 2^(m_s - M) acc_s / sum_s 2^(m_s - M) Z_s for head h of sequence b (head_dim a multiple
// of 4, at most 256).  Threads 0 .. 255 of the workgroup work -- a thread is (split lane, dim lane): it
// walks every SL-th partial with 16-byte loads, four of them in flight, and the split lanes are then
// added through LDS in a fixed order (a serial walk is bound by memory latency once a head has more
// than a handful of partials) -- but every thread of the workgroup must call: there are workgroup
// barriers inside.  seq_meta: the partials of sequence b are those of workgroups seq_meta[2b] ..
// + seq_meta[2b+1] of the one-pass focal kernel, wpk partials each.
template <typename T>
__device__ __forceinline__ void combine_wide_body(const float *__restrict__ part_o, const float *__restrict__ part_ml, int nsplit, int d,
                                                  T *__restrict__ out, float *__restrict__ lse, const int32_t *__restrict__ seq_meta,
                                                  int wpk, int h, int b, int Hq, const CombineShared<T> &sh)
{
    typedef typename CombineAcc<T>::type A;
    float *sm_max = sh.max4;
    A *sm_z = sh.z, *sm_o = sh.o;
    const int64_t bh = (int64_t)b * Hq + h;
    const int t = threadIdx.x;
    const bool works = t < 256;
    // partial s of this head: statistics at ml[s * ml_step], accumulator at po[s * o_step]
    const float *ml = part_ml + bh * nsplit * 2;
    const float *pbase = part_o + bh * nsplit * d;
    int64_t ml_step = 2, o_step = d;
    if (seq_meta) {
        const int64_t first = (int64_t)seq_meta[2 * b] * wpk;
        nsplit = seq_meta[2 * b + 1] * wpk;
        ml = part_ml + (first * Hq + h) * 2;
        pbase = part_o + (first * Hq + h) * d;
        ml_step = 2 * (int64_t)Hq;
        o_step = (int64_t)Hq * d;
    }
    // dim lanes: the power of two covering d/4 (1 .. 64); split lanes: the rest of the 256 threads
    const int nd4 = d / 4;
    int DL = 1;
    while (DL < nd4) DL <<= 1;
    const int SL = 256 / DL;
    const int dl = t & (DL - 1), sl = t / DL;
    const bool live = works && dl < nd4;          // this thread holds a (split lane, dim lane) of the merge

    A Z = 0;
    float M;
    typedef A Ax4 __attribute__((ext_vector_type(4)));
    Ax4 o = Ax4{0, 0, 0, 0};
    if (nsplit <= kCombineFew && nsplit <= 4 * SL) {
        // A handful of partials (a short list cut fine): one memory round trip instead of two.  The
        // thread's (at most four) accumulators are requested from clamped addresses, and by every
        // lane one of the maxima, which meet by lane moves instead of a reduction through LDS.  A loop over the maxima that every
        // thread reads is one scalar load and one wait per partial: hidden behind the accumulators up to a dozen of them (10 ranges, scores, mass and
        // merge of a warm-up layer: the layer 16.13 us against 16.37 by lanes), not beyond (32 ranges, dense attention 4 x 9216 tokens, 16/2 heads: 11.95 us
        // against 11.67; 16, a focal layer of 16 x 17152, 64/8: 194.0 against 191.4, head_dim 64 103.6 against 101.1).  From ten to sixteen the two are
        // within 0.5 us of each other (4608 tokens, 10 / 12 / 14 / 16 ranges, walk then lanes: dense attention, batch 4, 16/2 heads 11.29 / 10.44 /
        // 10.14 / 9.97, 11.91 / 10.80 / 10.50 / 10.16; 28/4 11.98 / 11.47 / 11.63 / 11.57, 12.33 / 11.86 / 11.89 / 11.82; 64/8 19.34 / 17.76 / 17.36 / 17.13,
        // 19.10 / 17.59 / 16.97 / 16.94; batch 12, 16/2 14.34 / 16.87 / 15.85 / 14.92, 14.28 / 16.63 / 15.59 / 14.68; a warm-up layer of them within 0.3).
        static_assert(kCombineFew <= 64, "a lane per partial");
        f32x4 a[4];
        float mm[4], zz[4];
        const int dc = dl < nd4 ? dl : nd4 - 1;
        const bool by_lane = nsplit > kCombineWalk;
        M = by_lane ? ml[min(t & 63, nsplit - 1) * ml_step] : -INFINITY;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int sk = sl + k * SL < nsplit ? sl + k * SL : 0;
            a[k] = *reinterpret_cast<const f32x4 *>(pbase + 4 * dc + sk * o_step);
            mm[k] = ml[sk * ml_step];
            zz[k] = ml[sk * ml_step + 1];
        }
        if (by_lane) {
            M = fmaxf(M, dpp_move<kDppXor1>(M));
            M = fmaxf(M, dpp_move<kDppXor2>(M));
            M = fmaxf(M, dpp_move<kDppHalfMirror>(M));
            M = fmaxf(rows_max(fmaxf(M, dpp_move<kDppRowMirror>(M))), -INFINITY);
        } else {
            for (int x = 0; x < nsplit; ++x) M = fmaxf(M, ml[x * ml_step]);
        }
        if (M > -INFINITY && live) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (sl + k * SL < nsplit) {
                    const A f = fast_exp2(mm[k] - M);
                    Z += f * zz[k];
                    o += __builtin_convertvector(a[k], Ax4) * f;
                }
            }
        }
    } else {
        float mloc = -INFINITY;
        if (works)
            for (int s = t; s < nsplit; s += 256) mloc = fmaxf(mloc, ml[s * ml_step]);
        mloc = wave_max(mloc);
        if (works && (t & 63) == 0) sm_max[t >> 6] = mloc;
        __syncthreads();
        M = fmaxf(fmaxf(sm_max[0], sm_max[1]), fmaxf(sm_max[2], sm_max[3]));
        if (M > -INFINITY && live) {
            const float *po = pbase + 4 * dl;
#pragma unroll 4
            for (int s = sl; s < nsplit; s += SL) {
                const A f = fast_exp2(ml[s * ml_step] - M);
                Z += f * ml[s * ml_step + 1];
                const f32x4 a = *reinterpret_cast<const f32x4 *>(po + s * o_step);
                o += __builtin_convertvector(a, Ax4) * f;
            }
        }
    }
    if (live) *reinterpret_cast<Ax4 *>(&sm_o[sl * d + 4 * dl]) = o;
    if (works && dl == 0) sm_z[sl] = Z;
    __syncthreads();
    if (t < d) {
        A acc = 0, zt = 0;
        for (int x = 0; x < SL; ++x) { acc += sm_o[x * d + t]; zt += sm_z[x]; }
        store_elem<T>(out + bh * d + t, zt > 0 ? (float)(acc / zt) : 0.f);
        if (lse && t == 0) lse[bh] = zt > 0 ? (M + log2f((float)zt)) * kLn2 : -INFINITY;
    }

}

// The image mass of sequence b: the sum of its partial sums, by one wave of a workgroup that has nothing else to do
// (a launch of its own took 1.5 us of the 27.6 us of a warm-up layer at batch 12, 4096 tokens, 16/2 heads).
__device__ __forceinline__ void image_mass_sum(const MassArgs &mass, const int32_t *__restrict__ seq_meta, int b)
{
    const int t = (int)threadIdx.x;
    if (t >= 64) return;
    const int64_t first = seq_meta ? seq_meta[2 * b] : (int64_t)b * mass.n_part;
    const int n = seq_meta ? seq_meta[2 * b + 1] : mass.n_part;
    float sum = 0.f;
    for (int x = t; x < n; x += 64) sum += mass.part[first + x];
    sum = wave_sum(sum);
    if (t == 0) mass.out[b] = sum;
}

}  // namespace fastocr
