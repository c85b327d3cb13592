"""The fp64 matrix-core kernels for fp32 caches (csrc/attn_f32.hip) against the oracle at the sizes where they can go
wrong: tile and range edges, group sizes up to the operand's width, uncut and cut lists, paged caches, every entry point."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_17447_amd as fo
from paper_2605_17447_amd import binding as fb
from util import TinyCase

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from gpu_util import DEV, GpuProblem, check_out, check_scores, paged_twin, problem_from_case, row_rel_err, to_np
    from test_gpu_parity import full_check


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Hq,Hkv", [(4, 1), (28, 4), (16, 1), (5, 5)])
def test_every_call_on_ragged_batches(Hq, Hkv, d):
    # lengths around a tile (16), a workgroup's round (64) and the uncut limit (128 / 192), one sequence long
    case = TinyCase(seed=50 + Hq, B=6, Hq=Hq, Hkv=Hkv, d=d, n_vis=[1, 15, 16, 49, 177, 2000], pre=[0, 1, 15, 0, 9, 33],
                    post=[1, 0, 17, 15, 7, 30], dtype="f32", spread=2.0)
    for tau in (0.05, 1.0):
        full_check(problem_from_case(case, "bhsd"), tau, f"f32 {Hq}/{Hkv} d={d} tau={tau}")
    full_check(problem_from_case(case, "bshd"), 0.05, "token-major")
    full_check(paged_twin(problem_from_case(case), 16, 3), 0.05, "paged, 16-token pages")
    full_check(paged_twin(problem_from_case(case), 24, 4), 0.05, "paged, pages that are no multiple of a tile")


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("nsplit", [1, 2, 7, 40])
def test_forced_range_counts(nsplit, d):
    case = TinyCase(seed=61, B=2, Hq=8, Hkv=2, d=d, n_vis=[900, 130], pre=[3, 20], post=[40, 1], dtype="f32")
    p = problem_from_case(case)
    try:
        for key in ("splits_score", "splits_dense", "splits_sparse"):
            fb.set_tuning(key, nsplit)
        full_check(p, 0.1, f"nsplit {nsplit}")
    finally:
        for key in ("splits_score", "splits_dense", "splits_sparse"):
            fb.set_tuning(key, 0)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("B,Hq,Hkv,merges", [(24, 8, 8, 1), (32, 8, 8, 1), (33, 8, 8, 1), (54, 8, 8, 1), (55, 8, 8, 0), (33, 16, 8, 0)])
def test_streams_that_fill_the_chip_unevenly_are_cut(B, Hq, Hkv, merges, d):
    # up to 256 streams are cut to fill the chip (192 of them in four), 257 to 435 of one query head each in three, more not at all
    n = [330 + 11 * (b % 7) for b in range(B)]
    case = TinyCase(seed=90 + B, B=B, Hq=Hq, Hkv=Hkv, d=d, n_vis=n, pre=[b % 5 for b in range(B)], post=[9 + b % 3 for b in range(B)], dtype="f32")
    p = problem_from_case(case)
    fb.kernel_timer_enable(fb.KERNEL_ATTN_COMBINE, 8)
    try:
        p.dense()
        got = len(fb.kernel_timer_read(fb.KERNEL_ATTN_COMBINE))
    finally:
        fb.kernel_timer_enable(fb.KERNEL_ATTN_COMBINE, 0)
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert got == merges
    full_check(p, 0.5, f"{B * Hkv} streams d={d}")


@pytest.mark.parametrize("d,n", [(64, 300), (128, 5000)])
def test_focal_layer_in_one_call_selects_like_the_separate_calls(d, n):
    case = TinyCase(seed=71, B=3, Hq=28, Hkv=4, d=d, n_vis=[n, n // 3, 0], pre=[5, 0, 4], post=[11, 70, 3], dtype="f32")
    p = problem_from_case(case)
    ref, _, ref_mass = oracle.focal_score(*p.oracle_args())
    dense, _ = oracle.decode_attn(*p.oracle_args())
    tau = 0.05
    kmax = fo.keep_count(p.batch.max_vis_len, tau)
    timers = (fb.KERNEL_FOCAL_FUSED, fb.KERNEL_DENSE_ATTN, fb.KERNEL_SCORE_LOGITS)
    results = []
    for mode in (1, 0):                                    # one pass; the separate calls
        fb.set_tuning("focal_fused", mode)
        for k in timers:
            fb.kernel_timer_enable(k, 8)
        try:
            out = torch.full_like(p.q, 3.0)
            sc = torch.zeros((p.B, p.batch.max_vis_len), dtype=torch.float32, device=DEV)
            idx = torch.zeros((p.B, kmax), dtype=torch.int32, device=DEV)
            cnt = torch.zeros((p.B,), dtype=torch.int32, device=DEV)
            mass = torch.zeros((p.B,), dtype=torch.float32, device=DEV)
            fo.focal_attn_score_topk(p.cache, p.batch, p.q, p.scale, tau, out, sc, idx, cnt,
                                     p.ws(fb.OP_FOCAL_ATTN_SCORE_TOPK, kmax), img_mass=mass)
            torch.cuda.synchronize()
            launches = tuple(len(fb.kernel_timer_read(k)) for k in timers)
        finally:
            fb.set_tuning("focal_fused", 1)
            for k in timers:
                fb.kernel_timer_enable(k, 0)
        assert launches == ((1, 0, 0) if mode else (0, 1, 1))
        results.append((to_np(sc), idx.cpu().numpy()))
        check_out(out, dense, f"mode {mode}")
        check_scores(sc, ref, p.vis_len, f"mode {mode}")
        assert np.abs(mass.cpu().numpy() - ref_mass).max() <= 1e-5
        for b in range(p.B):
            k = fo.keep_count(p.vis_len[b], tau)
            assert int(cnt[b]) == k
            want = oracle.topk(to_np(sc)[b, : p.vis_len[b]], k) if k else np.zeros(0, np.int32)
            assert np.array_equal(idx[b, :k].cpu().numpy(), want)
    # The logits are the same bits; the two forms cut the list into other ranges, so a head's sum differs by the roundings of
    # at most 42 partials merged in fp32 (a chain of up to 9 merges of 3 roundings, 2^-24 each): 1.6e-6 of a score.
    (one, one_idx), (apart, apart_idx) = results
    for b in range(p.B):
        m, k = p.vis_len[b], fo.keep_count(p.vis_len[b], tau)
        if k == 0:
            continue
        assert (np.abs(one[b, :m] - apart[b, :m]) <= 2e-6 * apart[b, :m]).all()
        last = apart[b, apart_idx[b, :k]].min()
        moved = np.setxor1d(one_idx[b, :k], apart_idx[b, :k])
        assert (np.abs(apart[b, moved] - last) <= 4e-6 * last).all(), "the sets differ by more than ties at the threshold"


def test_rows_that_are_not_16_byte_aligned_take_the_plain_kernels():
    # a cache whose base is 4 bytes off, and one whose token stride is odd: same results through the general path
    case = TinyCase(seed=81, B=2, Hq=8, Hkv=2, d=64, n_vis=[200, 90], pre=[3, 0], post=[5, 17], dtype="f32")
    p = problem_from_case(case)
    for shift, pad in ((1, 0), (0, 1)):
        B, H, S, d = p.k.shape
        kv = []
        for t in (p.k, p.v):
            raw = torch.zeros(B * H * S * (d + pad) + shift, dtype=t.dtype, device=t.device)
            view = torch.as_strided(raw, (B, H, S, d), (H * S * (d + pad), S * (d + pad), d + pad, 1), shift)
            view.copy_(t)
            kv.append(view)
        o = GpuProblem(kv[0], kv[1], p.q, p.seq_len, p.vis_start, p.vis_len, p.scale)
        got, _ = o.dense()
        want, _ = oracle.decode_attn(*p.oracle_args())
        check_out(got, want, f"shift {shift} pad {pad}")
        assert row_rel_err(got, p.dense()[0].double().cpu().numpy()) <= 1e-5
