// Focal layer in one pass (Sec. 3.1.1, Eq. 1; Alg. 1, focal branch): the layer's dense decode
// attention output AND the head-averaged focal scores of the image tokens from a single read
// of K and V.  A focal layer needs both -- its own attention output over the full cache and the
// scores that the following layers' fixation sets are cut from -- and K is the larger part of
// either computation's traffic, so reading it twice (dense attention, then scoring) wastes a
// third of the bytes.
//
// head_dim 128 and 64.  At 64 the tiles are half as large, so two tiles of K and of V are in flight per wave instead of one;
// batch 16, 16384 image tokens, 64/8 heads: 100 us for 563 MB (5.6 TB/s) where dense attention, its merge and scoring
// took 89 + 5 + 54 us and read K twice.
//
// Structure (shared with the scoring-only kernel in score_resident.hip):
//   - one 512-thread workgroup per (image-token range, sequence), at most one per compute unit,
//     so the whole grid is resident; wave w streams KV head w % Hkv in 32-token tiles;
//   - K and V tiles travel HBM -> LDS directly (one 8 KB slot each per wave); the next K tile is
//     requested as soon as the current one has been read into registers, likewise for V, so one
//     tile of each is always in flight while the other is being consumed;
//   - logits are produced transposed, C[token][column]: columns 0..7 are the group's heads for
//     the tile's first 16 tokens, columns 8..15 the same heads for its last 16 (two accumulators,
//     one select), so every lane holds 4 logits of ONE head.  Their softmax weights, which P*V needs anyway, stay in 4 VGPRs named
//     for the tile until the normalisers are known, relative to the running maximum of their time, which LDS keeps.  (Parked logits, whose
//     exponentials were taken behind the exchange, where nothing hides them, and lane moves of three instructions each: 64/8 heads,
//     16 x 16384, 6.2 us from the statistics to the sums over the heads, now 4.1);
//   - head_dim 64 has the registers and the idle matrix cores to produce the logits a second time with the operands exchanged,
//     C[head][token]: 4 heads of one token per lane, in the scoring kernel's arithmetic step by step, so that both kernels' scores
//     are the same bits and a set never depends on which of them a focal layer ran.  The sum over a token's heads is then four
//     products in the lane instead of lane moves (behind the exchange, 64/8 heads, 16 x 16384: 7 -> 2.7 us);
//   - the first layout serves P*V: with P masked to "first-half tokens in columns 0..7, second-half
//     tokens in columns 8..15" one v_mfma_f32_16x16x32_bf16 per 16 output dims accumulates
//     O^T[dim][column]; columns n and n+8 are the two halves' partial sums of head n and are added
//     at the end.  The running maximum of a head is uniform over the wave (it scales whole
//     accumulator columns); rescaling happens only in tiles where some head's maximum grew;
//   - each wave leaves an attention partial (accumulator, max, sum) in the workspace for the
//     split-merge kernel of attn.hip; the ranges then exchange their softmax statistics, meet at
//     the per-sequence barrier and turn the parked logits into scores exactly as the
//     scoring-only kernel does.
#include "kernels.hpp"
#include "resident.hpp"

namespace fastocr {

// statistics words per (workgroup, head), per sequence the count of ranges done reading, and a
// count of the waves that gave up waiting: same protocol as score_resident.hip, own arrays
__device__ unsigned long long g_fus_stats[kResSlots][kResMaxWg * kResMaxHq];
__device__ uint32_t g_fus_left[kResSlots][kResMaxBatch];
__device__ uint32_t g_fus_timeouts;
__device__ uint32_t g_fus_done[kResSlots][kResMaxBatch];     // fused top-k: ranges of a sequence whose scores are out

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
// One logit per image tile of the wave, indexed by the (wave-uniform) tile number: the compiler
// keeps such a vector in 32 consecutive VGPRs and addresses it through the register-index mode,
// so the tile loop stays a loop instead of 32 unrolled copies that overflow the instruction cache.
typedef float f32x32 __attribute__((ext_vector_type(32)));
static_assert(kResTmax == 32, "one f32x32 per logit row holds kResTmax tiles");

template <int D, bool PAGED, bool SELECT>
__global__ __launch_bounds__(kResThreads) void focal_fused_kernel(
    SelectArgs sel_args /* first: read straight from the kernel-argument segment when the select starts */,
    KvDev kv, BatchDev bv, const uint16_t *__restrict__ q, int Hq, int G, float scale_log2,
    int batch, int nranges_uniform, int R_uniform, int sync_slot, long long spin_ticks,
    float *__restrict__ scores, float *__restrict__ lse_out, float *__restrict__ mass_part,
    float *__restrict__ att_o, float *__restrict__ att_ml, int32_t *__restrict__ seq_meta,
    uint32_t *__restrict__ gave_up_flag)
{
    static_assert(sizeof(unsigned char[kResWaves][2][8192]) >= (size_t)kSelLdsBytes, "the select reuses the tile buffers");
    __shared__ __align__(256) unsigned char smem[kResWaves][2][8192];     // [wave][K, V][slot]

    static_assert(D == 128 || D == 64, "head_dim 128 or 64");
    constexpr int KS = D / 32;             // k-steps of a logit
    constexpr int NACC = D / 16;           // 16-dim blocks of the output
    constexpr int NL = D / 16;             // 1 KB load instructions per 32-token K (or V) tile
    constexpr int RPL = 32 / NL;           // rows one load instruction brings
    constexpr int CPR = D / 8;             // 16-byte chunks of a row
    constexpr int ROWB = 2 * D;            // bytes of a row
    constexpr int NSLOT = 128 / D;         // tiles of K (and of V) in flight: 8 KB each way, whatever the head_dim
    constexpr int NV = D == 128 ? 4 : 2;   // distinct chunk permutations over the loads of a K tile
    __shared__ float sm_m[kResWaves][8], sm_z[kResWaves][8];
    __shared__ __align__(16) float sm_ref[D == 128 ? kResWaves : 1][kResTmax][8];
    __shared__ float sm_red[kResWaves];
    __shared__ int sm_met, sm_last;

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int li = lane & 15, lg = lane >> 4;                      // the lane in the matrix products
    const int lrow = lane / CPR, lslot = lane % CPR;               // the lane in a load: row of the load's group, chunk slot in LDS
    const int Hkv = kv.n_kv_heads;
    const int wpk = kResWaves / Hkv;
    const int kvh = wave % Hkv, sub = wave / Hkv;

    // which sequence and which of its ranges (all wave-uniform); ragged batches get ranges in
    // proportion to their lengths
    const RangeAlloc ra = resident_alloc(bv, batch, gridDim.x, nranges_uniform, R_uniform, kResTile * wpk, blockIdx.x);
    if (!ra.active) return;
    const int rng = ra.rng, b = ra.b, nranges = ra.nr, R = ra.R, wg0 = ra.wg0;
    const int S = ra.S, v0 = ra.v0, N = ra.N;
    // where the sequence's partials are, for the merge and image-mass kernels that follow
    if (rng == 0 && threadIdx.x == 0) { seq_meta[2 * b] = wg0; seq_meta[2 * b + 1] = nranges; }
    const int Tn = S - N;

    // image tiles of this wave: tile ti = sub + j*wpk of the range, j = 0 .. nimg-1
    const int r0 = rng * R, r1 = min(N, r0 + R);
    const int nt_range = r1 > r0 ? (r1 - r0 + kResTile - 1) / kResTile : 0;
    const int nimg = min(nt_range > sub ? (nt_range - sub + wpk - 1) / wpk : 0, kResTmax);
    // text tiles of this wave: u = slot + i*nslots
    const int ntt = (Tn + kResTile - 1) / kResTile;
    const int slot = rng * wpk + sub, nslots = nranges * wpk;
    const int ntext = ntt > slot ? (ntt - slot + nslots - 1) / nslots : 0;

    // Q as the B operand of the logits: column n = li holds head n & 7 of the group
    const int hcol = li & 7;
    const bool hi = li >= 8;                     // this lane's logits belong to the tile's last 16 tokens
    u32x4 qq[KS];
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
        qq[kk] = u32x4{0u, 0u, 0u, 0u};
        if (hcol < G)
            qq[kk] = *reinterpret_cast<const u32x4 *>(q + ((int64_t)b * Hq + (int64_t)kvh * G + hcol) * D + 8 * (4 * kk + lg));
    }
    const uint16_t *kbase = reinterpret_cast<const uint16_t *>(kv.k);
    const uint16_t *vbase = reinterpret_cast<const uint16_t *>(kv.v);

    const int rot = nimg > 0 ? (wave * 5 + rng * 3 + b * 7) % nimg : 0;
    auto img_first = [&](int x) {                                                  // span-relative
        int j = x + rot;
        j = j >= nimg ? j - nimg : j;
        return r0 + (sub + j * wpk) * kResTile;
    };
    auto text_first = [&](int x) { return (slot + x * nslots) * kResTile; };       // text-relative

    // Tile number n of the wave goes into slot n % NSLOT of its K and V buffers: load e brings rows RPL e ..
    // RPL e + RPL - 1, lane (lrow, lslot) one 16-byte chunk of row r = RPL e + lrow, which lands at slot + 1024 e +
    // 16 lane.  For K the chunk is lslot ^ f(r), f(r) = r & 15 (D 128) or (r >> 1) & 7 (D 64): the swizzle that
    // makes the MFMA operand reads conflict-free; V stays row-major (chunk lslot).  Rows past the end of a
    // ragged tile are clamped to its last row.
    const int64_t seq_base = row_offset<false>(kv, b, 0, kvh);
    const uint32_t stride_b = (uint32_t)kv.stride_token * 2u;            // bytes; 32 rows fit 32 bits (host-checked)
    const uint32_t rowoff_row = (uint32_t)lrow * stride_b;
    const int fl = D == 128 ? lrow : (lrow >> 1);
    const uint32_t chunk_k0 = 16u * (uint32_t)(lslot ^ fl);
    // (the permutations differ by an exclusive or with 4 (e & NV - 1) chunks; formed where they are used, they would live in registers
    // that the loop does not have)
    auto chunk_k = [&](int e) { return chunk_k0 ^ (uint32_t)(64 * (e & (NV - 1))); };
    const uint32_t chunk_v = 16u * (uint32_t)lslot;
    const unsigned char *kbytes = reinterpret_cast<const unsigned char *>(kv.k);
    const unsigned char *vbytes = reinterpret_cast<const unsigned char *>(kv.v);

    auto slot_of = [&](int n, bool isv) { return smem[wave][isv ? 1 : 0] + (n & (NSLOT - 1)) * (8192 / NSLOT); };
    auto issue_run = [&](int first_tok, int rv, int n, bool isv) {
        unsigned char *dst = slot_of(n, isv);
        const unsigned char *bytes = isv ? vbytes : kbytes;
        const uint32_t limit = (uint32_t)(rv - 1) * stride_b;
        if (PAGED) {
            const int pt = kv.page_tokens;
            const int pg0 = first_tok / pt, in0 = first_tok - pg0 * pt;
            const int32_t *bt = kv.block_table + (int64_t)b * kv.max_pages;
            const int64_t pa = bt[min(pg0, kv.max_pages - 1)], pb = bt[min(pg0 + 1, kv.max_pages - 1)];
            const unsigned char *base_a = bytes + 2 * (pa * kv.stride_page + (int64_t)kvh * kv.stride_head + (int64_t)in0 * kv.stride_token);
            const unsigned char *base_b = bytes + 2 * (pb * kv.stride_page + (int64_t)kvh * kv.stride_head + (int64_t)(in0 - pt) * kv.stride_token);
            const uint32_t split = (uint32_t)(pt - in0) * stride_b;      // first byte offset of the second page
#pragma unroll
            for (int e = 0; e < NL; ++e) {
                const uint32_t ro = min(rowoff_row + (uint32_t)(RPL * e) * stride_b, limit);
                const unsigned char *base = ro >= split ? base_b : base_a;
                lds_dma16(reinterpret_cast<const uint16_t *>(base + (ro + (isv ? chunk_v : chunk_k(e)))), dst + 1024 * e);
            }
        } else {
            const unsigned char *base = bytes + 2 * (seq_base + (int64_t)first_tok * kv.stride_token);
#pragma unroll
            for (int e = 0; e < NL; ++e) {
                const uint32_t ro = min(rowoff_row + (uint32_t)(RPL * e) * stride_b, limit);
                lds_dma16(reinterpret_cast<const uint16_t *>(base + (ro + (isv ? chunk_v : chunk_k(e)))), dst + 1024 * e);
            }
        }
    };
    // Past the wave's last tile the refill stays unconditional (the readers' counts of outstanding
    // loads rely on it) but fetches one row of the query, which is in cache.
    const uint16_t *qrow = q + ((int64_t)b * Hq + (int64_t)kvh * G) * D;
    auto issue_dummy = [&](int n, bool isv) {
        unsigned char *dst = slot_of(n, isv);
#pragma unroll
        for (int e = 0; e < NL; ++e) lds_dma16(qrow + chunk_v / 2, dst + 1024 * e);
    };
    auto issue_img = [&](int x, bool isv) {
        if (x >= nimg) { issue_dummy(ntext + x, isv); return; }
        const int jf = img_first(x);
        issue_run(v0 + jf, min(kResTile, r1 - jf), ntext + x, isv);
    };
    // text positions map to tokens with a gap at the image span, so the rows are addressed one by one
    auto issue_text = [&](int x, bool isv) {
        const int tf = text_first(x);
        unsigned char *dst = slot_of(x, isv);
        const uint16_t *base = isv ? vbase : kbase;
#pragma unroll
        for (int e = 0; e < NL; ++e) {
            const int tc = min(tf + RPL * e + lrow, Tn - 1);
            const int tok = tc < v0 ? tc : tc + N;
            lds_dma16(base + row_offset<PAGED>(kv, b, tok, kvh) + (isv ? chunk_v : chunk_k(e)) / 2, dst + 1024 * e);
        }
    };
    // tile number n of the wave (text tiles first, then image tiles), or the dummy past the end
    auto issue_any = [&](int n, bool isv) {
        if (n < ntext) issue_text(n, isv);
        else issue_img(n - ntext, isv);
    };

    const int tt0 = 16 * (li >> 3) + 4 * lg;        // tile-relative token of this lane's first logit
    // Running max, uniform over the head's lanes (lane li: head li & 7).  Head_dim 128: z is this lane's sum; the weights
    // parked so far stay as they are when m grows -- there are no registers to bring 128 of them along -- and m is noted in LDS for
    // every image tile; bit J of moved_at says that it grew there (or that tile J is the first).
    float m = kMinusHuge, z = 0.f;
    uint32_t moved_at = 1u;
    // Head_dim 64: the scoring kernel's references and sums (score_resident.hip) of heads 4 (lg & 1) .. + 3, this lane's token of a tile
    const int tok_in_tile = li + 16 * (lg >> 1);
    float ref[4] = {kMinusHuge, kMinusHuge, kMinusHuge, kMinusHuge}, zr[4] = {0.f, 0.f, 0.f, 0.f};
    f32x32 park0, park1, park2, park3;              // the weight of token r (D 64: head r) of the lane in image tile J: park<r>[J]
    f32x4 acc[NACC];
#pragma unroll
    for (int t = 0; t < NACC; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};

    // LDS byte addresses in slot 0: K rows li and 16 + li as the A operand, V rows 4lg.. and 16 + 4lg..
    // (chunk 4 kk + lg of a row, permuted: an exclusive or with 64 kk bytes)
    const uint32_t rd_k = lds_address(&smem[wave][0][0]) + li * ROWB + (((lg ^ (D == 128 ? li : (li >> 1))) & (CPR - 1)) << 4);
    const uint32_t rd_v = lds_address(&smem[wave][1][0]) + (4 * lg) * ROWB + (li & (CPR - 1)) * 16;

    // Loads are sent in the order K(n), V(n), K(n+1), ..; when K(n) is wanted the newest ones outstanding
    // are V(n) and, with two slots, K(n+1) and V(n+1); when V(n) is wanted, K and V of the tiles between
    // and the K refill just sent: 8 loads with one slot (D 128), 12 with two (D 64), so "at most that many
    // outstanding" means the tile has landed.  Reads and waits are written in assembly: the compiler
    // neither orders LDS reads after loads that land in LDS by themselves without draining ALL of them, nor
    // may it move the products above the wait.
    // rows li (first call) and 16 + li (second call) of the K tile, in two halves so that only
    // four operand registers are live at a time
    auto read_k_lo = [&](uint32_t so, u32x4(&kb)[KS]) {
        if constexpr (D == 64)
            asm volatile(
                "s_waitcnt vmcnt(12)\n\t"
                "ds_read_b128 %0, %2\n\t"
                "ds_read_b128 %1, %3\n\t"
                "s_waitcnt lgkmcnt(0)"
                : "=&v"(kb[0]), "=&v"(kb[1])
                : "v"(rd_k + so), "v"((rd_k ^ 64u) + so)
                : "memory");
        else asm volatile(
            "s_waitcnt vmcnt(8)\n\t"
            "ds_read_b128 %0, %4\n\t"
            "ds_read_b128 %1, %5\n\t"
            "ds_read_b128 %2, %6\n\t"
            "ds_read_b128 %3, %7\n\t"
            "s_waitcnt lgkmcnt(0)"
            : "=&v"(kb[0]), "=&v"(kb[1]), "=&v"(kb[2]), "=&v"(kb[3])
            : "v"(rd_k), "v"(rd_k ^ 64u), "v"(rd_k ^ 128u), "v"(rd_k ^ 192u)
            : "memory");
    };
    auto read_k_hi = [&](uint32_t so, u32x4(&kb)[KS]) {
        if constexpr (D == 64)
            asm volatile(
                "ds_read_b128 %0, %2 offset:2048\n\t"
                "ds_read_b128 %1, %3 offset:2048\n\t"
                "s_waitcnt lgkmcnt(0)"
                : "=&v"(kb[0]), "=&v"(kb[1])
                : "v"(rd_k + so), "v"((rd_k ^ 64u) + so)
                : "memory");
        else asm volatile(
            "ds_read_b128 %0, %4 offset:4096\n\t"
            "ds_read_b128 %1, %5 offset:4096\n\t"
            "ds_read_b128 %2, %6 offset:4096\n\t"
            "ds_read_b128 %3, %7 offset:4096\n\t"
            "s_waitcnt lgkmcnt(0)"
            : "=&v"(kb[0]), "=&v"(kb[1]), "=&v"(kb[2]), "=&v"(kb[3])
            : "v"(rd_k), "v"(rd_k ^ 64u), "v"(rd_k ^ 128u), "v"(rd_k ^ 192u)
            : "memory");
    };
    // vv[e]: chunk li (D 64: li & 7) of the row of token 4lg + e (e < 4) or 16 + 4lg + e - 4 of the tile
    auto read_v = [&](uint32_t so, u32x4(&vv)[8]) {
        if constexpr (D == 64)
            asm volatile(
                "s_waitcnt vmcnt(12)\n\t"
                "ds_read_b128 %0, %8\n\t"
                "ds_read_b128 %1, %8 offset:128\n\t"
                "ds_read_b128 %2, %8 offset:256\n\t"
                "ds_read_b128 %3, %8 offset:384\n\t"
                "ds_read_b128 %4, %8 offset:2048\n\t"
                "ds_read_b128 %5, %8 offset:2176\n\t"
                "ds_read_b128 %6, %8 offset:2304\n\t"
                "ds_read_b128 %7, %8 offset:2432\n\t"
                "s_waitcnt lgkmcnt(0)"
                : "=&v"(vv[0]), "=&v"(vv[1]), "=&v"(vv[2]), "=&v"(vv[3]), "=&v"(vv[4]), "=&v"(vv[5]), "=&v"(vv[6]), "=&v"(vv[7])
                : "v"(rd_v + so)
                : "memory");
        else asm volatile(
            "s_waitcnt vmcnt(8)\n\t"
            "ds_read_b128 %0, %8\n\t"
            "ds_read_b128 %1, %8 offset:256\n\t"
            "ds_read_b128 %2, %8 offset:512\n\t"
            "ds_read_b128 %3, %8 offset:768\n\t"
            "ds_read_b128 %4, %8 offset:4096\n\t"
            "ds_read_b128 %5, %8 offset:4352\n\t"
            "ds_read_b128 %6, %8 offset:4608\n\t"
            "ds_read_b128 %7, %8 offset:4864\n\t"
            "s_waitcnt lgkmcnt(0)"
            : "=&v"(vv[0]), "=&v"(vv[1]), "=&v"(vv[2]), "=&v"(vv[3]), "=&v"(vv[4]), "=&v"(vv[5]), "=&v"(vv[6]), "=&v"(vv[7])
            : "v"(rd_v)
            : "memory");
    };

    // One tile: logits, online softmax, P*V.  nlive = tokens of the tile that exist (may exceed 32).  Returns the weights to park.
    auto tile_step = [&](int n, int nlive, auto &&next_k, auto &&next_v) -> f32x4 {
        f32x4 weights;
        const uint32_t so = (uint32_t)(n & (NSLOT - 1)) * (8192 / NSLOT);
        u32x4 kb[KS];
        f32x4 c0 = f32x4{0.f, 0.f, 0.f, 0.f}, c1 = c0, t0 = c0, t1 = c0;
        read_k_lo(so, kb);
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) {
            c0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kb[kk]),
                                                         __builtin_bit_cast(bf16x8, qq[kk]), c0, 0, 0, 0);
            if constexpr (D == 64)
                t0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, qq[kk]),
                                                             __builtin_bit_cast(bf16x8, kb[kk]), t0, 0, 0, 0);
        }
        read_k_hi(so, kb);
        next_k();
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) {
            c1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kb[kk]),
                                                         __builtin_bit_cast(bf16x8, qq[kk]), c1, 0, 0, 0);
            if constexpr (D == 64)
                t1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, qq[kk]),
                                                             __builtin_bit_cast(bf16x8, kb[kk]), t1, 0, 0, 0);
        }
        if constexpr (D == 64) {
            const bool live = tok_in_tile < nlive;
            f32x4 w;
            bool moved = false;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float x = lg >= 2 ? t1[r] : t0[r];
                w[r] = live ? x * scale_log2 : -INFINITY;
                if (ref[r] == kMinusHuge) ref[r] = fmaxf(w[r], kMinusHuge);          // the first live logit
                moved = moved || w[r] - ref[r] > kRefSlack;
            }
            if (__builtin_amdgcn_ballot_w64(moved) != 0ull) {
                float a[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const bool mv = w[r] - ref[r] > kRefSlack;
                    a[r] = mv ? fast_exp2(ref[r] - w[r]) : 1.f;
                    ref[r] = mv ? w[r] : ref[r];
                    zr[r] *= a[r];
                }
                // (tile by tile: as whole vectors they would be copied)
                for (int x = 0; x < n - ntext; ++x) {
                    park0[x] *= a[0];
                    park1[x] *= a[1];
                    park2[x] *= a[2];
                    park3[x] *= a[3];
                }
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                w[r] = fast_exp2(w[r] - ref[r]);
                zr[r] += w[r];
            }
            weights = w;
        }
        float p[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float x = hi ? c1[r] : c0[r];
            p[r] = (tt0 + r < nlive) ? x * scale_log2 : -INFINITY;
        }
        float mx = fmaxf(fmaxf(p[0], p[1]), fmaxf(p[2], p[3]));
        mx = fmaxf(mx, dpp_move<kDppRor8>(mx));
        mx = rows_max(mx);
        const float m_new = fmaxf(m, mx);
        if (__builtin_amdgcn_ballot_w64(m_new != m) != 0ull) {
            const float alpha = fast_exp2(m - m_new);
#pragma unroll
            for (int t = 0; t < NACC; ++t) acc[t] *= alpha;
            if constexpr (D == 128) {
                z *= alpha;
                if (n >= ntext) moved_at |= 1u << (n - ntext);
            }
            m = m_new;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) p[r] = fast_exp2(p[r] - m);
        if constexpr (D == 128) {
            z += (p[0] + p[1]) + (p[2] + p[3]);
            weights = f32x4{p[0], p[1], p[2], p[3]};
        }
        const uint32_t w0 = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)p[0], (__bf16)p[1]});
        const uint32_t w1 = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)p[2], (__bf16)p[3]});
        // contraction slots of lane group lg: tokens 4lg..4lg+3, then 16+4lg..16+4lg+3
        const u32x4 pb = u32x4{hi ? 0u : w0, hi ? 0u : w1, hi ? w0 : 0u, hi ? w1 : 0u};

        u32x4 vv[8];
        read_v(so, vv);
        next_v();
#pragma unroll
        for (int t = 0; t < NACC; ++t) {
            // D 128: row i of block t is dim 8i + t; D 64: rows i and i + 8 share chunk i & 7 and take its even and
            // odd elements, dim 8 (i & 7) + 2t + (i >> 3)
            const int w = D == 128 ? t >> 1 : t;
            const uint32_t selb = (D == 128 ? (t & 1) != 0 : hi) ? 0x07060302u : 0x05040100u;
            u32x4 a;
#pragma unroll
            for (int pp = 0; pp < 4; ++pp) a[pp] = __builtin_amdgcn_perm(vv[2 * pp + 1][w], vv[2 * pp][w], selb);
            acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                             __builtin_bit_cast(bf16x8, pb), acc[t], 0, 0, 0);
        }
        return weights;
    };

    // ---- stream: text tiles, then image tiles (weights parked in registers) ----------------------
    if (ntext + nimg > 0) {
        issue_any(0, false);
        issue_any(0, true);
        if constexpr (NSLOT == 2) { issue_any(1, false); issue_any(1, true); }
        for (int x = 0; x < ntext; ++x)
            (void)tile_step(x, Tn - text_first(x), [&]() { issue_any(x + NSLOT, false); }, [&]() { issue_any(x + NSLOT, true); });
        for (int J = 0; J < nimg; ++J) {
            const f32x4 w = tile_step(ntext + J, r1 - img_first(J), [&]() { issue_img(J + NSLOT, false); }, [&]() { issue_img(J + NSLOT, true); });
            park0[J] = w[0];
            park1[J] = w[1];
            park2[J] = w[2];
            park3[J] = w[3];
            if constexpr (D == 128) sm_ref[wave][J][hcol] = m;
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // the trailing refills must not land later

    // Lane coordinates are derived afresh for the rest of the kernel: carried across the tile loop
    // they would occupy registers it has no room for.
    int tx_p = threadIdx.x;
    asm volatile("" : "+v"(tx_p));
    const int lane_p = tx_p & 63, li_p = lane_p & 15, lg_p = lane_p >> 4, hcol_p = li_p & 7, hbase_p = 4 * (lg_p & 1);

    // ---- the wave's statistics per head: what the weights are relative to, and their sum ----------------------
    if constexpr (D == 128) {
        z += dpp_move<kDppRor8>(z);
        z = rows_sum(z);
        if (lane_p < 8) { sm_m[wave][lane_p] = m; sm_z[wave][lane_p] = z; }
    } else {
        // in the scoring kernel's steps and roundings
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float M = ref[r];
            M = fmaxf(M, dpp_move<kDppXor1>(M));
            M = fmaxf(M, dpp_move<kDppXor2>(M));
            M = fmaxf(M, dpp_move<kDppHalfMirror>(M));
            M = fmaxf(M, dpp_move<kDppRowMirror>(M));
            M = with_lane_xor32(M, [](float a, float b) { return fmaxf(a, b); });
            const float e = fast_exp2(ref[r] - M);
            float Z = fmaf(zr[r], e, dpp_move<kDppXor1>(zr[r] * e));
            Z += dpp_move<kDppXor2>(Z);
            Z += dpp_move<kDppHalfMirror>(Z);
            Z += dpp_move<kDppRowMirror>(Z);
            Z = with_lane_xor32(Z, [](float a, float b) { return a + b; });
            if (li_p == 0 && lg_p < 2) { sm_m[wave][hbase_p + r] = M; sm_z[wave][hbase_p + r] = Z; }
        }
        wave_lds_fence();
        // relative to the running maximum, as the partial has it (a reference lies at most kRefSlack below)
        z = sm_z[wave][li_p & 7] * fast_exp2(sm_m[wave][li_p & 7] - m);
    }

    // ---- attention partial of this wave: O^T columns n and n + 8 are the same head's halves -----
#pragma unroll
    for (int t = 0; t < NACC; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[t][r] += dpp_move<kDppRor8>(acc[t][r]);
    if constexpr (D == 64) {
        // operand row 4lg + r: lane groups 0 and 1 hold the even dims of chunks 4 (lg & 1) + r, groups 2 and 3 the odd
        // ones; after the half swaps acc[0..3][r] are four consecutive dims of the chunk, its first four in
        // groups 0 and 1, its last four in groups 2 and 3
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float x[4];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                // (copies: a bit cast of a vector element itself reads element 0)
                const float even = acc[t][r], later = acc[t + 2][r];
                const auto sw = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, even), __builtin_bit_cast(uint32_t, later),
                                                                 false, false);
                x[2 * t] = __builtin_bit_cast(float, (uint32_t)sw[0]);
                x[2 * t + 1] = __builtin_bit_cast(float, (uint32_t)sw[1]);
            }
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[t][r] = x[t];
        }
    }
    if (li_p < 8 && li_p < G) {
        const int64_t row = ((int64_t)(wg0 + rng) * wpk + sub) * Hq + kvh * G + li_p;      // [workgroup][sub][head]
        if constexpr (D == 128) {
            // lane_p (head li_p, group lg_p) holds dims 32lg + 8r + t in acc[t][r]
            float *po = att_o + row * 128 + 32 * lg_p;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                *reinterpret_cast<f32x4 *>(po + 8 * r) = f32x4{acc[0][r], acc[1][r], acc[2][r], acc[3][r]};
                *reinterpret_cast<f32x4 *>(po + 8 * r + 4) = f32x4{acc[4][r], acc[5][r], acc[6][r], acc[7][r]};
            }
        } else {
            float *po = att_o + row * 64 + 32 * (lg_p & 1) + 4 * (lg_p >> 1);
#pragma unroll
            for (int r = 0; r < 4; ++r)
                *reinterpret_cast<f32x4 *>(po + 8 * r) = f32x4{acc[0][r], acc[1][r], acc[2][r], acc[3][r]};
        }
        if (lg_p == 0) {
            att_ml[2 * row] = m;
            att_ml[2 * row + 1] = z;
        }
    }
    if (threadIdx.x == 0) sm_met = 1;
    __syncthreads();

    // ---- range statistics: published as self-validating words, gathered by polling (resident.hpp) ----
    // (Asking for the other ranges' words before the partial is written, as the scoring kernel does at the
    // end of its stream, gains 0.4 us at the largest shapes and loses 2 us at the small ones, where the
    // ranges end together, the first answer comes back incomplete and a second round trip follows.)
    unsigned long long *stats = g_fus_stats[sync_slot] + (int64_t)wg0 * Hq;
    resident_publish(stats + (int64_t)rng * Hq, sm_m, sm_z, Hq, G, Hkv, wpk);
    // (reference, sum) of this wave's heads over the whole sequence (lane 8s + x: head x of the group)
    float Mh, Zh;
    {
        const bool ok = resident_heads_gather<4>(stats, rng, nranges, Hq, G, Hkv, wpk, kvh, sm_m, sm_z, spin_ticks, Mh, Zh);
        if (!ok && lane_p == 0) {
            sm_met = 0;
            __hip_atomic_fetch_add(&g_fus_timeouts, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (gave_up_flag) __hip_atomic_store(gave_up_flag, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
    __syncthreads();      // whether every wave has met its ranges
    // This range is done reading: count it out.  The last one of the sequence clears the
    // sequence's words and the count when the kernel ends.
    uint32_t *left = &g_fus_left[sync_slot][b];
    // (the count's old value is only looked at when the kernel ends: nobody waits for the atomic)
    uint32_t left_before = 0u;
    if (threadIdx.x == 0) left_before = __hip_atomic_fetch_add(left, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    auto leave = [&]() {
        if (threadIdx.x == 0) sm_last = left_before == (uint32_t)nranges - 1u;
        __syncthreads();
        resident_retire(sm_last != 0, stats, nranges, Hq, left);
    };
    if (!sm_met) {
        // a range of the sequence never published: poison this range's scores
        for (int i = threadIdx.x; i < r1 - r0; i += kResThreads)
            store_score<SELECT>(&scores[(int64_t)b * bv.max_vis_len + r0 + i], __builtin_nanf(""));
        if (SELECT) resident_select_tail(scores, b, nranges, &g_fus_done[sync_slot][b], &smem[0][0][0]);
        leave();
        return;
    }
    if (lse_out && rng == 0 && sub == 0 && lane_p < G) lse_out[(int64_t)b * Hq + kvh * G + lane_p] = resident_lse(Mh, Zh);

    // ---- the parked weights brought to the normalisers, summed over the heads of each token: one row of sums per four heads,
    // [2 Hkv][R], at most 64 KB -----------------------------------------------------------------------
    float *red = reinterpret_cast<float *>(&smem[0][0][0]);
    if constexpr (D == 128) {
        const float Mx = __shfl(Mh, hcol_p), ix = 1.0f / __shfl(Zh, hcol_p);
        const float Mc = hcol_p < G ? Mx : INFINITY, ic = hcol_p < G ? ix : 0.f;
        float c = 0.f;
        float *to = red + (2 * kvh + ((li_p >> 2) & 1)) * R - r0 + 16 * (li_p >> 3) + 4 * lg_p + (li_p & 3);
        const bool odd = (li_p & 1) != 0, high = (li_p & 2) != 0;
#pragma unroll 2
        for (int J = 0; J < nimg; ++J) {
#pragma clang fp contract(off)
            if ((moved_at >> J) & 1u) c = fast_exp2(sm_ref[wave][J][hcol_p] - Mc) * ic;
            // 4 tokens of tile J in each of 4 neighbouring lanes, a head each: lane k ends up with the sum of token k
            const float v0 = park0[J] * c, v1 = park1[J] * c, v2 = park2[J] * c, v3 = park3[J] * c;
            const float y0 = (odd ? v1 : v0) + dpp_move<kDppXor1>(odd ? v0 : v1);
            const float y1 = (odd ? v3 : v2) + dpp_move<kDppXor1>(odd ? v2 : v3);
            to[img_first(J)] = (high ? y1 : y0) + dpp_move<kDppXor2>(high ? y0 : y1);
        }
    } else {
        float cf[4];
        resident_factors(Mh, Zh, ref, hbase_p, G, cf);
        float *to = red + (2 * kvh + (lg_p & 1)) * R - r0 + li_p + 16 * (lg_p >> 1);
        for (int J = 0; J < nimg; ++J) {
            const f32x4 w = f32x4{park0[J], park1[J], park2[J], park3[J]};
            to[img_first(J)] = resident_head_sum(w, cf);
        }
    }
    __syncthreads();
    // Where the rest of the kernel starts in a 64-byte instruction line makes up to 1.2 us of difference at a few tiles per wave (it
    // runs once, on all compute units at about the same time, after a stream that leaves little of it in the caches), so its
    // start is fixed at byte 36, whatever comes before it.  Measured in steps of 4 and 8 bytes, 36 to 44 are best in all forms of
    // the kernel (36 by up to 0.5 us with one sequence); us with the merge's launch at byte 4 / 20 / 36 / 52: 12/2 heads, batch 8, 3000 image tokens, head_dim 128
    // 21.2 / 21.1 / 20.4 / 21.2, 64 17.5 / 17.5 / 16.5 / 17.5; 28/4 heads, batch 10, 1392 image tokens 23.1 / 22.6 / 22.3 / 23.0 and
    // 18.3 / 17.6 / 17.3 / 18.2; 64/8 heads, batch 16, 16384: no difference.
    asm volatile(".p2align 6\n\t.rept 9\n\ts_nop 0\n\t.endr");
    float local = 0.f;
    const float inv = 1.0f / (float)Hq;
    const int rows = 2 * Hkv;
    for (int i = threadIdx.x; i < r1 - r0; i += kResThreads) {
        float a = 0.f;
        for (int g = 0; g < rows; ++g) a += red[g * R + i];
        a *= inv;
        store_score<SELECT>(&scores[(int64_t)b * bv.max_vis_len + r0 + i], a);
        local += a;
    }
    if (mass_part) {
        local = wave_sum(local);
        if (lane_p == 0) sm_red[wave] = local;
        __syncthreads();
        if (threadIdx.x == 0) {
            float t = 0.f;
            for (int w = 0; w < kResWaves; ++w) t += sm_red[w];
            mass_part[wg0 + rng] = t;
        }
    }
    if (SELECT) resident_select_tail(scores, b, nranges, &g_fus_done[sync_slot][b], &smem[0][0][0]);
    leave();
}

// Workspace, with W = nranges * batch workgroups: attention partials fp32 [W][wpk][Hq][d] and
// [W][wpk][Hq][2], image-mass partials [W], and per sequence
// its first workgroup and range count int32 [B][2].
// Sized for the most workgroups that this or a smaller problem's plan can have: a plan's own count goes up and
// down as its range length is rounded, and a size asked for once has to serve shorter sequences as well.
size_t focal_fused_workspace_bytes(const Shape &s, int num_cu)
{
    const size_t W = (size_t)resident_max_workgroups(s, num_cu);
    if (W == 0) return 0;
    const size_t wpk = (size_t)(kResWaves / s.kv.n_kv_heads);
    size_t bytes = W * wpk * s.n_q_heads * (s.kv.head_dim + 2) * sizeof(float);
    bytes += W * sizeof(float);
    bytes += (size_t)s.batch * 2 * sizeof(int32_t);
    return bytes;
}

hipError_t focal_fused_timeouts(uint32_t *n) { return hipMemcpyFromSymbol(n, HIP_SYMBOL(g_fus_timeouts), sizeof(uint32_t)); }

hipError_t launch_focal_fused(const Shape &s, const ResidentPlan &p, int sync_slot, uint32_t *flag, const void *q, float scale,
                              void *out, float *scores, float *lse, float *img_mass, void *ws, hipStream_t stream,
                              const SelectArgs *select, CombineArgs *defer)
{
    if (sync_slot < 0 || sync_slot >= kResSlots) return hipErrorInvalidValue;
    const int W = p.nranges * s.batch;
    float *att_o = reinterpret_cast<float *>(ws);
    float *att_ml = att_o + (size_t)W * p.wpk * s.n_q_heads * s.kv.head_dim;
    float *mass_part = att_ml + (size_t)W * p.wpk * s.n_q_heads * 2;
    int32_t *seq_meta = reinterpret_cast<int32_t *>(mass_part + W);
    const float scale_log2 = scale * kLog2e;
    const int G = s.n_q_heads / s.kv.n_kv_heads;
    const long long spin_ticks = tune_spin_ticks();                  // 0.25 s unless overridden

    dim3 grid(W), block(kResThreads);
    const bool fuse = select && select->sel_idx;
    if (fuse && !resident_select_fits(s)) return hipErrorInvalidValue;
    const SelectArgs sa = fuse ? *select : SelectArgs{0.0, nullptr, nullptr, nullptr, nullptr, 0};
#define FASTOCR_FUS(D, P, S) FASTOCR_LAUNCH(K_FOCAL_FUSED, (focal_fused_kernel<D, P, S>), grid, block, 0, stream, sa, s.kv, s.bv, \
                       (const uint16_t *)q, s.n_q_heads, G, scale_log2, s.batch, p.nranges, p.range_tokens, \
                       sync_slot, spin_ticks, scores, lse, img_mass ? mass_part : nullptr, att_o, att_ml, seq_meta, flag)
#define FASTOCR_FUS_D(D) \
    if (s.paged) { if (fuse) FASTOCR_FUS(D, true, true); else FASTOCR_FUS(D, true, false); } \
    else         { if (fuse) FASTOCR_FUS(D, false, true); else FASTOCR_FUS(D, false, false); }
    if (s.kv.head_dim == 64) { FASTOCR_FUS_D(64) } else { FASTOCR_FUS_D(128) }
#undef FASTOCR_FUS_D
#undef FASTOCR_FUS
    const MassArgs mass{mass_part, img_mass, 0};          // summed by the launch that merges the output's partials
    // every sequence's partials: workgroups seq_meta[b][0] .. + seq_meta[b][1], wpk of them each
    if (defer) {
        *defer = CombineArgs{att_o, att_ml, p.nranges * p.wpk, s.kv.head_dim, s.n_q_heads, p.wpk, seq_meta, out, false, mass};
        return hipGetLastError();
    }
    return launch_attn_combine(s, att_o, att_ml, p.nranges * p.wpk, out, nullptr, stream, seq_meta, p.wpk, mass);
}

}  // namespace fastocr
