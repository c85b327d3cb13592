// Decode attention and focal scoring over fp32 caches on the fp64 matrix cores (gfx950).
//
// The fp32 outputs are held to 1e-5 of their row maximum whatever the logits' size, so the q.k sums, the weight
// sums and the p.V sums run in fp64.  On the matrix cores: v_mfma_f64_16x16x4_f64, tokens on one side and the
// G = Hq/Hkv query heads that share a kv head on the other, so that every K and V row is read once per kv head
// (the one-wave-per-query-head kernels of attn.hip and score.hip read it G times and are bound by chains of
// fp64 FMAs behind per-lane row walks).
//   QK^T : A = K tile (16 tokens x 4 dims), B = Q^T  -> C[token][head]
//   PV   : A = V^T (16 dims x 4 tokens),    B = P^T  -> C[dim][head]
// An operand holds one fp64 value per lane: lane (li, lg) = (lane % 16, lane / 16) has row li, contraction index lg; C
// has row 4r + lg in element r of lane (li, lg), column li.  So C of the first product, read with r as the
// step and lg as the contraction index, IS the B operand of the second, and the contraction order over dims
// is free as long as K and Q agree:
//   K : lane (li, lg) loads dims 16c + 4 lg .. +3 of token li (16 bytes; 64 contiguous bytes per row and load), step
//       (c, e) contracts the four dims 16c + 4 lg + e;
//   V : lane (li, lg) loads dims 64h + 4 li .. +3 of token 4r + lg (whole 256-byte pieces of a row), block (h, e)
//       has dim 64h + 4i + e in its row i.
// Both arrive in operand order straight from memory: no LDS, no transposition, one conversion per element.
//
// Bound: HBM; per 16 tokens and kv head a wave spends D/2 matrix instructions (64 cycles each), at head_dim 128
// 28 us of matrix time next to 40 us of bytes for 4 sequences x 16704 tokens x 4 kv heads.  Two waves per SIMD
// (<= 256 registers: Q and the accumulators take 64 each as fp64, a K and a V tile 32 each): while
// one waits for its tile or takes exponentials the other one's products run; a wave asks for its next K tile as
// soon as the present one is consumed, likewise for V.  Measured at that size (28 query heads, 273 MB): 272 -> 51 us
// (1.0 -> 5.4 TB/s) for dense attention.  Q in LDS and the registers used for a second K tile: 56 us.
#include "kernels.hpp"
#include "combine.hpp"

namespace fastocr {

typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int kF32Tile = 16;       // tokens per wave tile
constexpr int kF32Waves = 4;
constexpr double kRound = 6755399441055744.0;      // 1.5 * 2^52

__device__ __forceinline__ f32x4 stream_load_f32(const float *p)
{
    return __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(p));
}

// One workgroup per (token range, kv head, sequence); the attended list is cut into nsplit * kF32Waves pieces of
// whole tiles, one per wave.  PV: attention output (DIRECT: the final one, else an fp32 partial).
// PARK: the logits (log2 domain, rounded to fp32 once) go to logits[b][kvh][token][Gp] for score_finalize_kernel.
// part_ml gets the range's (max, sum-exp) per head in either case.
template <int D, bool GATHER, bool PAGED, bool DIRECT, bool PV, bool PARK>
__global__ __launch_bounds__(64 * kF32Waves, 2) void attn_f32_kernel(
    const int32_t *__restrict__ seq_len, const int32_t *__restrict__ vis_start, const int32_t *__restrict__ vis_len,
    const int32_t *__restrict__ sel_cnt, const int32_t *__restrict__ sel_idx, int64_t kmax, int nsplit,
    KvDev kv, int max_seq_len, int max_vis_len, const float *__restrict__ q, int Hq, int G, double scale_log2,
    float *__restrict__ part_o, float *__restrict__ part_ml, float *__restrict__ out,
    float *__restrict__ lse, float *__restrict__ logits, int64_t pitch)
{
    static_assert(D == 128 || D == 64, "head_dim 128 or 64");
    static_assert(PV || PARK, "something to compute");
    static_assert(!(GATHER && PARK), "scores are those of the whole cache");
    constexpr int NC = D / 16;            // 16-byte pieces of a K row per lane
    constexpr int NH = D / 64;            // 256-byte pieces of a V row
    __shared__ __align__(16) double sm_o[PV ? kF32Waves : 1][PV ? D * 16 : 1];
    __shared__ float sm_m[kF32Waves][16];
    __shared__ double sm_z[kF32Waves][16];

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int li = lane & 15, lg = lane >> 4;
    const int split = blockIdx.x, kvh = blockIdx.y, b = blockIdx.z;

    const BatchDev bv{seq_len, vis_start, vis_len, max_seq_len, max_vis_len};
    const int nw = nsplit * kF32Waves;
    // Gather: tiles dealt in turn, to all workgroups' first waves before their second ones, and the set first in the list, so that the entries of
    // a wave's first three tiles are asked for together with the lengths (the pointers are in registers when a wave starts): two round
    // trips before the first row instead of four (4/1 heads of 64, 45 attended tokens: 5.0 -> 4.4 us in the kernel).
    const int gw = GATHER ? wave * nsplit + split : split * kF32Waves + wave;
    const int32_t *sel = GATHER ? sel_idx + (int64_t)b * kmax : nullptr;
    const int s_len = seq_len[b], v_start = vis_start[b], v_len = vis_len[b], s_cnt = GATHER ? sel_cnt[b] : 0;
    int entry[3] = {0, 0, 0};
    if (GATHER) {
#pragma unroll
        for (int i = 0; i < 3; ++i) entry[i] = sel[min((int64_t)((gw + i * nw) * kF32Tile + li), kmax - 1)];
    }
    asm volatile("" :: "s"(s_len), "s"(v_start), "s"(v_len), "s"(s_cnt), "s"(kv.k), "s"(kv.v), "s"(kv.stride_token), "s"(kv.stride_head),
                 "s"(kv.stride_seq), "s"(q), "s"(Hq), "s"(G), "s"(max_seq_len), "s"(max_vis_len) : "memory");
    const SeqGeom geo = seq_geom_of(bv, s_len, v_start, v_len);
    const int cnt = GATHER ? min(max(s_cnt, 0), (int)min((int64_t)geo.N, kmax)) : 0;
    const int L = GATHER ? (geo.S - geo.N + cnt) : geo.S;
    const int ntile = (L + kF32Tile - 1) / kF32Tile;
    // else piece gw starts at tile floor(gw * ntile / nw): the pieces that hold a tile more are spread over the workgroups
    const int x = ntile / nw, rem = ntile - x * nw;
    const int u0 = GATHER ? gw : gw * x + gw * rem / nw;
    const int nt = GATHER ? x + (gw < rem ? 1 : 0) : (gw + 1) * x + (gw + 1) * rem / nw - u0;
    const int wp0 = u0 * kF32Tile, wstep = GATHER ? nw * kF32Tile : kF32Tile, pend = GATHER ? L : min(L, (u0 + nt) * kF32Tile);

    // Q as the B operand: lane (head li, lg) holds dims 16c + 4 lg + e for step (c, e); lanes past the group's heads its last one again
    double qd[NC][4];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const f32x4 v = *reinterpret_cast<const f32x4 *>(q + ((int64_t)b * Hq + (int64_t)kvh * G + min(li, G - 1)) * D + 16 * c + 4 * lg);
#pragma unroll
        for (int e = 0; e < 4; ++e) qd[c][e] = (double)v[e];
    }

    const float *kbase = reinterpret_cast<const float *>(kv.k);
    const float *vbase = reinterpret_cast<const float *>(kv.v);
    const int64_t seq_base = row_offset<false>(kv, b, 0, kvh);
    // Row look-up of tile i for token li, in stages of one load each; a stage's load is sent a tile ahead of
    // its use and before that tile's rows, so that waiting for it never waits for rows (loads return in order).
    auto pos_of = [&](int i, int row) { return min(wp0 + i * wstep + row, pend - 1); };
    auto slot_load = [&](int i) -> int { return GATHER ? sel[min(pos_of(i, li), max(cnt - 1, 0))] : 0; };
    auto token_of = [&](int i, int raw) -> int {
        const int p = pos_of(i, li);
        if (!GATHER) return p;
        const int mid = geo.v0 + min(max(raw, 0), max(geo.N - 1, 0)), t = p - cnt;
        return t < 0 ? mid : (t < geo.v0 ? t : t + geo.N);
    };
    auto page_load = [&](int tok) -> int {
        return PAGED ? kv.block_table[(int64_t)b * kv.max_pages + min((int)((uint32_t)tok / (uint32_t)kv.page_tokens), kv.max_pages - 1)] : 0;
    };
    auto offset_of = [&](int tok, int page) -> int64_t {
        if (!PAGED) return seq_base + (int64_t)tok * kv.stride_token;
        const int in = tok - (int)((uint32_t)tok / (uint32_t)kv.page_tokens) * kv.page_tokens;
        return (int64_t)page * kv.stride_page + (int64_t)in * kv.stride_token + (int64_t)kvh * kv.stride_head;
    };

    f32x4 K[NC], V[PV ? 4 : 1][NH];
    auto issue_k = [&](int64_t off) {
#pragma unroll
        for (int c = 0; c < NC; ++c) K[c] = stream_load_f32(kbase + off + 16 * c + 4 * lg);
    };
    auto issue_v = [&](int i, int64_t off) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            int64_t ro;
            if (GATHER || PAGED) ro = __shfl(off, 4 * r + lg);
            else ro = seq_base + (int64_t)pos_of(i, 4 * r + lg) * kv.stride_token;
#pragma unroll
            for (int h = 0; h < NH; ++h) V[r][h] = stream_load_f32(vbase + ro + 64 * h + 4 * li);
        }
    };

    // Running maximum of head li: an fp32 value, exact as a double.  It starts finite, so that a tile of keys that are all
    // masked out (logits of -inf, or below the type's lowest value) leaves weights of 0 behind, not of 2^(inf - inf).
    float m = kLowest;
    double z = 0.0;                      // this lane's share of head li's weight sum
    f64x4 acc[PV ? 4 * NH : 1];
    if constexpr (PV) {
#pragma unroll
        for (int t = 0; t < 4 * NH; ++t) acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
    }
    const int Gp = (G + 3) / 4 * 4;
    float *lpark = PARK ? logits + ((int64_t)b * kv.n_kv_heads + kvh) * pitch * Gp + li : nullptr;

    if (nt > 0) {
        if (GATHER && geo.S == geo.N) {              // no text: rows past the end are to repeat the set's last one, never another
#pragma unroll
            for (int i = 0; i < 3; ++i) entry[i] = slot_load(i);
        }
        int tok1 = token_of(0, entry[0]);
        int64_t off0 = offset_of(tok1, page_load(tok1));
        tok1 = token_of(1, entry[1]);
        int page1 = page_load(tok1), raw2 = entry[2];
        issue_k(off0);
        if constexpr (PV) issue_v(0, off0);
        for (int i = 0; i < nt; ++i) {
            f64x4 s0 = f64x4{0.0, 0.0, 0.0, 0.0}, s1 = s0;
#pragma unroll
            for (int c = 0; c < NC; ++c) {
#pragma unroll
                for (int e = 0; e < 4; e += 2) {
                    s0 = __builtin_amdgcn_mfma_f64_16x16x4f64((double)K[c][e], qd[c][e], s0, 0, 0, 0);
                    s1 = __builtin_amdgcn_mfma_f64_16x16x4f64((double)K[c][e + 1], qd[c][e + 1], s1, 0, 0, 0);
                }
            }
            // tile i + 1: its token and page entry are there; tile i + 2: its entry of the set is
            const int64_t off1 = offset_of(tok1, page1);
            tok1 = token_of(i + 2, raw2);
            page1 = page_load(tok1);
            raw2 = slot_load(i + 3);
            issue_k(off1);
            // lane (head li, lg): s[r] is token 4r + lg of the tile
            double s[4];
            float mx = -INFINITY;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                s[r] = (s0[r] + s1[r]) * scale_log2;
                const float f = (wp0 + i * wstep + 4 * r + lg < pend) ? (float)s[r] : -INFINITY;
                mx = fmaxf(mx, f);
                if (PARK && li < Gp) lpark[(int64_t)(wp0 + i * wstep + 4 * r + lg) * Gp] = f;      // inside the pitch
            }
            mx = rows_max(mx);
            // a whole number: the factors between maxima, here and where waves and ranges are merged, are then exact
            // powers of two instead of exponentials off by an ulp each
            const float m_new = fmaxf(m, ceilf(mx));
            if (__builtin_amdgcn_ballot_w64(m_new != m) != 0ull) {
                const double alpha = (double)fast_exp2(m - m_new);
                z *= alpha;
                if constexpr (PV) {
#pragma unroll
                    for (int t = 0; t < 4 * NH; ++t) acc[t] *= alpha;
                }
                m = m_new;
            }
            // The weight from the exact difference, its whole part apart: fp32 holds the rest to 2^-25, where the
            // difference itself (10 and more octaves for most tokens of a flat distribution) would be rounded to 2^-21.
            // Rounded by adding and taking off 1.5 * 2^52, whose low word then holds the whole part: defined for every
            // value, where the conversion to an integer is not.  Below -2000 the weight is 0 in fp64 anyway and
            // taken as that: a logit of -inf has no whole part and no rest.  A NaN passes and stays one.
            double p[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const double x = s[r] - (double)m, y = x + kRound, whole = y - kRound;
                const double w = ldexp((double)fast_exp2((float)(x - whole)), (int)(uint32_t)__builtin_bit_cast(uint64_t, y));
                p[r] = (wp0 + i * wstep + 4 * r + lg < pend) && !(x < -2000.0) ? w : 0.0;
                z += p[r];
            }
            if constexpr (PV) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int h = 0; h < NH; ++h)
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            acc[4 * h + e] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)V[r][h][e], p[r], acc[4 * h + e], 0, 0, 0);
                issue_v(i + 1, off1);
            }
        }
    }

    // ---- lanes -> wave -> workgroup -------------------------------------------------------------
    z += __shfl_xor(z, 16);
    z += __shfl_xor(z, 32);
    if (lg == 0) { sm_m[wave][li] = m; sm_z[wave][li] = z; }
    __syncthreads();
    float M = sm_m[0][li];
#pragma unroll
    for (int w = 1; w < kF32Waves; ++w) M = fmaxf(M, sm_m[w][li]);
    if constexpr (PV) {
        const double f = M > -INFINITY ? (double)fast_exp2(m - M) : 0.0;
#pragma unroll
        for (int t = 0; t < 4 * NH; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) sm_o[wave][(4 * t + r) * 64 + lane] = acc[t][r] * f;
        __syncthreads();
        double Z = 0.0;
        if (M > -INFINITY) {
#pragma unroll
            for (int w = 0; w < kF32Waves; ++w) Z += (double)fast_exp2(sm_m[w][li] - M) * sm_z[w][li];
        }
        // thread -> (h, r) of its lane: four consecutive dims 64h + 4 (4r + lg) .. +3 of head li
        const int64_t bh = (int64_t)b * Hq + (int64_t)kvh * G + li;
#pragma unroll
        for (int u = 0; u < NH * 4 / kF32Waves; ++u) {
            const int hr = wave + kF32Waves * u, h = hr >> 2, r = hr & 3;
            if (li >= G) continue;
            f32x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                double a = 0.0;
#pragma unroll
                for (int w = 0; w < kF32Waves; ++w) a += sm_o[w][(4 * (4 * h + e) + r) * 64 + lane];
                o[e] = DIRECT ? (Z > 0.0 ? (float)(a / Z) : 0.f) : (float)a;
            }
            const int dim = 64 * h + 4 * (4 * r + lg);
            if (DIRECT) *reinterpret_cast<f32x4 *>(out + bh * D + dim) = o;
            else *reinterpret_cast<f32x4 *>(part_o + (bh * nsplit + split) * D + dim) = o;
        }
        if (wave == 0 && lg == 0 && li < G) {
            if (DIRECT) {
                if (lse) lse[bh] = Z > 0.0 ? (M + log2f((float)Z)) * kLn2 : -INFINITY;
            } else {
                part_ml[(bh * nsplit + split) * 2] = M;
                part_ml[(bh * nsplit + split) * 2 + 1] = (float)Z;
            }
        }
    } else {
        if (wave == 0 && lg == 0 && li < G) {
            double Z = 0.0;
            if (M > -INFINITY) {
#pragma unroll
                for (int w = 0; w < kF32Waves; ++w) Z += (double)fast_exp2(sm_m[w][li] - M) * sm_z[w][li];
            }
            const int64_t bh = (int64_t)b * Hq + (int64_t)kvh * G + li;
            part_ml[(bh * nsplit + split) * 2] = M;
            part_ml[(bh * nsplit + split) * 2 + 1] = (float)Z;
        }
    }
}

// sel_idx: pruned attention; logits: the logits are parked as well; part_o == nullptr and out == nullptr: nothing but that.
// nsplit == 1 with `out` and without `logits`: the kernel writes the final output itself.
hipError_t launch_attn_f32(int kid, const Shape &s, const void *q, float scale, const int32_t *sel_idx, const int32_t *sel_cnt,
                           int64_t kmax, float *part_o, float *part_ml, int nsplit, void *out, float *lse, float *logits,
                           int64_t pitch, hipStream_t stream)
{
    const int G = s.n_q_heads / s.kv.n_kv_heads;
    dim3 grid(nsplit, s.kv.n_kv_heads, s.batch), block(64 * kF32Waves);
    const double scale_log2 = (double)scale * 1.4426950408889634074;     // unrounded
    const bool pv = part_o != nullptr, direct = pv && !logits && nsplit == 1;
#define FASTOCR_F32K(D, GA, PG, DI, PV, PK) FASTOCR_LAUNCH(kid, (attn_f32_kernel<D, GA, PG, DI, PV, PK>), grid, block, 0, stream, \
        s.bv.seq_len, s.bv.vis_start, s.bv.vis_len, sel_cnt, sel_idx, kmax, nsplit, s.kv, s.bv.max_seq_len, s.bv.max_vis_len, \
        (const float *)q, s.n_q_heads, G, scale_log2, part_o, part_ml, (float *)out, lse, logits, pitch)
#define FASTOCR_F32D(D, PG) \
    if (sel_idx) { if (direct) FASTOCR_F32K(D, true, PG, true, true, false); else FASTOCR_F32K(D, true, PG, false, true, false); } \
    else if (!pv) FASTOCR_F32K(D, false, PG, false, false, true); \
    else if (logits) FASTOCR_F32K(D, false, PG, false, true, true); \
    else if (direct) FASTOCR_F32K(D, false, PG, true, true, false); \
    else FASTOCR_F32K(D, false, PG, false, true, false)
    if (s.kv.head_dim == 64) { if (s.paged) { FASTOCR_F32D(64, true); } else { FASTOCR_F32D(64, false); } }
    else                     { if (s.paged) { FASTOCR_F32D(128, true); } else { FASTOCR_F32D(128, false); } }
#undef FASTOCR_F32D
#undef FASTOCR_F32K
    return hipGetLastError();
}

}  // namespace fastocr
