"""The last launch of a focal layer with its top-k: the select shares it with the merge of the output's partials, with and
without the image mass, and gives the bits of the separate calls."""
import pytest
import torch

import paper_2605_17447_amd as fo
from paper_2605_17447_amd import binding as fb
from util import TinyCase

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from gpu_util import DEV, problem_from_case


def _layer(p, tau, mass):
    kmax = fo.keep_count(p.batch.max_vis_len, tau)
    out, sc = torch.full_like(p.q, 3.0), torch.full((p.B, p.batch.max_vis_len), -7.0, dtype=torch.float32, device=DEV)
    idx, cnt = torch.full((p.B, kmax), -1, dtype=torch.int32, device=DEV), torch.full((p.B,), -1, dtype=torch.int32, device=DEV)
    fo.focal_attn_score_topk(p.cache, p.batch, p.q, p.scale, tau, out, sc, idx, cnt, p.ws(fb.OP_FOCAL_ATTN_SCORE_TOPK, kmax), img_mass=mass)
    return out, sc, idx, cnt


@pytest.fixture(params=[1, 2], ids=["by size", "single kernel"])
def fused(request):
    """The library's choice, which parks the logits at these sizes, and the one-pass kernel (fp32 caches: the same form twice)."""
    fb.set_tuning("focal_fused", request.param)
    yield request.param
    fb.set_tuning("focal_fused", 1)


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 64)])
@pytest.mark.parametrize("B,apart", [(20, 0), (21, 1)])          # 1280 and 1344 merges of 64 heads, 256 compute units
def test_many_merges_keep_their_own_launch(dtype, d, B, apart, fused):
    n = [40 + 7 * (b % 9) for b in range(B)]
    case = TinyCase(seed=700 + d + B, B=B, Hq=64, Hkv=8, d=d, n_vis=n, pre=[b % 5 for b in range(B)], post=[b % 11 for b in range(B)], dtype=dtype)
    p = problem_from_case(case)
    tau = 0.1
    want_out, want_sc, _, want_mass = p.focal_attn(want_mass=True)
    want_idx, want_cnt = p.topk(want_sc, tau)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    fb.kernel_timer_enable(fb.KERNEL_ATTN_COMBINE, 16)
    try:
        for mass in (None, torch.full((B,), -3.0, dtype=torch.float32, device=DEV)):
            out, sc, idx, cnt = _layer(p, tau, mass)
            # (parked logits: the launch that finishes the scores merges the output where the select's does not)
            own = 0 if dtype == "bf16" and fused == 1 else apart if cus == 256 else int(64 * B > 5 * cus)
            assert len(fb.kernel_timer_read(fb.KERNEL_ATTN_COMBINE)) == own
            assert torch.equal(out, want_out) and torch.equal(cnt, want_cnt) and (mass is None or torch.equal(mass, want_mass))
            for b in range(B):
                assert torch.equal(sc[b, : n[b]], want_sc[b, : n[b]])
                assert torch.equal(idx[b, : int(cnt[b])], want_idx[b, : int(cnt[b])])
    finally:
        fb.kernel_timer_enable(fb.KERNEL_ATTN_COMBINE, 0)


@pytest.mark.parametrize("dtype,d,Hq,Hkv,B", [("bf16", 128, 28, 4, 3), ("bf16", 64, 64, 8, 5), ("bf16", 128, 8, 1, 40),
                                              ("f32", 128, 28, 4, 3), ("f32", 64, 4, 1, 7)])
def test_the_image_mass_is_summed_by_the_shared_launch(dtype, d, Hq, Hkv, B, fused):
    # ragged, one sequence without an image, one of a single image token; up to several partials of mass per sequence
    n = [(997 * (b + 1)) % 2300 + 3 for b in range(B)]
    n[1], n[2] = 0, 1
    case = TinyCase(seed=500 + d + B, B=B, Hq=Hq, Hkv=Hkv, d=d, n_vis=n, pre=[b % 5 for b in range(B)],
                    post=[40 + b for b in range(B)], dtype=dtype)
    p = problem_from_case(case)
    tau = 0.05
    want_out, want_sc, _, want_mass = p.focal_attn(want_mass=True)
    want_idx, want_cnt = p.topk(want_sc, tau)
    for k in (fb.KERNEL_ATTN_COMBINE, fb.KERNEL_TOPK):
        fb.kernel_timer_enable(k, 16)
    try:
        for with_mass in (False, True):
            mass = torch.full((B,), -3.0, dtype=torch.float32, device=DEV) if with_mass else None
            out, sc, idx, cnt = _layer(p, tau, mass)
            assert len(fb.kernel_timer_read(fb.KERNEL_ATTN_COMBINE)) == 0, "a merge launch of its own"
            assert len(fb.kernel_timer_read(fb.KERNEL_TOPK)) == 1
            assert torch.equal(out, want_out) and torch.equal(cnt, want_cnt)
            for b in range(B):
                assert torch.equal(sc[b, : n[b]], want_sc[b, : n[b]])
                assert torch.equal(idx[b, : int(cnt[b])], want_idx[b, : int(cnt[b])])
            if with_mass:
                assert torch.equal(mass, want_mass)
    finally:
        for k in (fb.KERNEL_ATTN_COMBINE, fb.KERNEL_TOPK):
            fb.kernel_timer_enable(k, 0)
