"""The one-pass focal kernel at head_dim 64 (128-byte rows, two tiles of K and of V in flight per wave) against the
oracle: one and several tiles per wave, more text than image, both layouts and paged, every kv head count it takes."""
import numpy as np
import pytest
import torch

import fastocr_synth as fs
import oracle
import paper_2605_17447_amd as fo
from paper_2605_17447_amd import binding as fb
from util import TinyCase

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from gpu_util import DEV, GpuProblem, check_out, check_scores, problem_from_case, to_np


def _check(p, what, tau=0.05):
    oc = p.oracle_args()
    ref_sc, ref_lse, ref_mass = oracle.focal_score(*oc)
    ref_dense, _ = oracle.decode_attn(*oc)
    fb.kernel_timer_read(fb.KERNEL_FOCAL_FUSED)
    fb.kernel_timer_enable(fb.KERNEL_PARKED_FINISH, 8)
    out, sc, lse, mass = p.focal_attn(want_lse=True, want_mass=True)
    assert len(fb.kernel_timer_read(fb.KERNEL_FOCAL_FUSED)) == 1, "the one-pass kernel did not run"
    assert len(fb.kernel_timer_read(fb.KERNEL_PARKED_FINISH)) == 0, "the logits were parked"
    fb.kernel_timer_enable(fb.KERNEL_PARKED_FINISH, 0)
    check_out(out, ref_dense, what)
    check_scores(sc, ref_sc, p.vis_len, what)
    assert np.allclose(lse.cpu().numpy(), ref_lse, rtol=2e-5, atol=2e-5)
    assert np.allclose(mass.cpu().numpy(), ref_mass, atol=2e-5)
    # the scoring kernel's scores, bit for bit: which of the two ran never changes a set
    alone, alone_lse, alone_mass = p.scores(want_lse=True, want_mass=True)
    for b, n in enumerate(p.vis_len):
        assert torch.equal(alone[b, :n], sc[b, :n]), f"{what}: sequence {b}'s scores differ from the scoring kernel's"
    assert torch.equal(alone_lse, lse) and torch.equal(alone_mass, mass)
    # with the top-k: the same output and scores bit for bit, and the exact set of these scores
    kmax = max(1, fo.keep_count(p.batch.max_vis_len, tau))
    out2, sc2 = torch.full_like(p.q, 3.0), torch.full_like(sc, -7.0)
    idx = torch.zeros((p.B, kmax), dtype=torch.int32, device=DEV)
    cnt = torch.zeros((p.B,), dtype=torch.int32, device=DEV)
    fo.focal_attn_score_topk(p.cache, p.batch, p.q, p.scale, tau, out2, sc2, idx, cnt, p.ws(fb.OP_FOCAL_ATTN_SCORE_TOPK, kmax))
    assert torch.equal(out, out2) and torch.equal(sc, sc2)
    for b, n in enumerate(p.vis_len):
        k = fo.keep_count(n, tau)
        assert int(cnt[b]) == k and np.array_equal(idx[b, :k].cpu().numpy(), oracle.topk(to_np(sc)[b, :n], k))


@pytest.mark.parametrize("Hq,Hkv", [(64, 8), (28, 4), (16, 2), (5, 1)])
def test_one_pass_focal_layer_head_dim_64(Hq, Hkv):
    fb.set_tuning("focal_fused", 2)
    fb.set_tuning("score_resident", 2)
    fb.kernel_timer_enable(fb.KERNEL_FOCAL_FUSED, 8)
    try:
        many = TinyCase(seed=900 + Hq, B=24, Hq=Hq, Hkv=Hkv, d=64, n_vis=[1500 + 61 * i for i in range(24)],
                        pre=[i % 7 * 5 for i in range(24)], post=[(i * 13) % 90 for i in range(24)], dtype="bf16")
        for layout in ("bhsd", "bshd"):
            _check(problem_from_case(many, layout), f"d64 {Hq}/{Hkv} {layout}")
        few = TinyCase(seed=901 + Hq, B=3, Hq=Hq, Hkv=Hkv, d=64, n_vis=[64, 200, 33], pre=[3000, 1500, 0],
                       post=[500, 2100, 4000], dtype="bf16", spread=2.0)
        _check(problem_from_case(few), f"d64 {Hq}/{Hkv} long text")
        steep = TinyCase(seed=903 + Hq, B=2, Hq=Hq, Hkv=Hkv, d=64, n_vis=[2000, 700], pre=[9, 0], post=[3, 100], dtype="bf16", spread=6.0)
        _check(problem_from_case(steep), f"d64 {Hq}/{Hkv} logits far above the first ones")
        one = TinyCase(seed=902 + Hq, B=2, Hq=Hq, Hkv=Hkv, d=64, n_vis=[31, 1], pre=[0, 0], post=[0, 1], dtype="bf16")
        _check(problem_from_case(one), f"d64 {Hq}/{Hkv} one tile", tau=0.25)
        wl = fs.config(5, batch=12, steps=4, n_visual=(600, 3000), grid_w=(20, 60), text_prefix=(3, 300), page_tokens=64,
                       head_dim=64, n_q_heads=Hq, n_kv_heads=Hkv)
        bt = fs.make_batch(wl, device=DEV)
        q = fs.queries_for_step(bt, 3, [x[2] for x in fs.centres(bt)])
        _check(GpuProblem(bt.k, bt.v, q, bt.seq_len(3), bt.vis_start, bt.n_vis, wl.head_dim ** -0.5, block_table=bt.block_table),
               f"d64 {Hq}/{Hkv} paged")
    finally:
        fb.kernel_timer_enable(fb.KERNEL_FOCAL_FUSED, 0)
        fb.set_tuning("focal_fused", 1)
        fb.set_tuning("score_resident", 1)


@pytest.mark.parametrize("d", [64, 128])
def test_scoring_kept_off_the_waiting_grid_keeps_the_head_dim_64_layer_off_it(d):
    case = TinyCase(seed=950, B=2, Hq=28, Hkv=4, d=d, n_vis=[900, 2000], pre=[9, 0], post=[3, 100], dtype="bf16")
    p = problem_from_case(case)
    want, _ = oracle.decode_attn(*p.oracle_args())
    ref_sc, _, _ = oracle.focal_score(*p.oracle_args())
    fb.kernel_timer_enable(fb.KERNEL_FOCAL_FUSED, 8)
    fb.set_tuning("focal_fused", 2)                              # (left to its size the layer would wait for nobody)
    try:
        for scoring, launches in ((1, 1), (0, 0 if d == 64 else 1)):
            fb.set_tuning("score_resident", scoring)
            out, sc, _, _ = p.focal_attn()
            assert len(fb.kernel_timer_read(fb.KERNEL_FOCAL_FUSED)) == launches, f"score_resident {scoring}"
            check_out(out, want, f"score_resident {scoring}")
            check_scores(sc, ref_sc, p.vis_len, f"score_resident {scoring}")
    finally:
        fb.kernel_timer_enable(fb.KERNEL_FOCAL_FUSED, 0)
        fb.set_tuning("focal_fused", 1)
        fb.set_tuning("score_resident", 1)
