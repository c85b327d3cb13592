"""The forms that park a bf16 cache's logits for a second launch (scoring, a focal layer, with and without the top-k) against the
oracle: tile, block and range edges, every way the heads are dealt, spans that start anywhere, dead keys, replays."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_17447_amd as fo
from paper_2605_17447_amd import binding as fb
from util import TinyCase, as_f64, f32_to_bf16_bits

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from gpu_util import DEV, GpuProblem, check_out, check_scores, paged_twin, problem_from_case, to_np


@pytest.fixture
def finish_launches():
    for k in (fb.KERNEL_PARKED_FINISH, fb.KERNEL_ATTN_COMBINE):
        fb.kernel_timer_enable(k, 64)
    yield lambda k: len(fb.kernel_timer_read(k))
    for k in (fb.KERNEL_PARKED_FINISH, fb.KERNEL_ATTN_COMBINE):
        fb.kernel_timer_enable(k, 0)


def _check(p, launches, what, ref=None, tau=0.07):
    """ref: (scores, lse, image mass, output) instead of the oracle's."""
    if ref is None:
        oc = p.oracle_args()
        ref = (*oracle.focal_score(*oc), oracle.decode_attn(*oc)[0])
    ref_sc, ref_lse, ref_mass, ref_out = ref
    sc, lse, mass = p.scores(want_lse=True, want_mass=True)
    assert launches(fb.KERNEL_PARKED_FINISH) == 1, what
    check_scores(sc, ref_sc, p.vis_len, what + " scores")
    assert np.allclose(lse.cpu().numpy(), ref_lse, rtol=2e-5, atol=2e-5) and np.allclose(mass.cpu().numpy(), ref_mass, atol=2e-5), what
    for b, n in enumerate(p.vis_len):
        assert (sc[b, n:] == -7.0).all(), f"{what}: scores past sequence {b}'s image were written"
    out, sc, lse, mass = p.focal_attn(want_lse=True, want_mass=True)
    assert launches(fb.KERNEL_ATTN_COMBINE) == 0 and launches(fb.KERNEL_PARKED_FINISH) == 1, what      # one launch for all of it
    check_out(out, ref_out, what + " output")
    check_scores(sc, ref_sc, p.vis_len, what + " layer's scores")
    assert np.allclose(lse.cpu().numpy(), ref_lse, rtol=2e-5, atol=2e-5) and np.allclose(mass.cpu().numpy(), ref_mass, atol=2e-5), what
    # with the top-k, in launches of its own and inside: the same bits, the exact set of these scores
    kmax = max(1, fo.keep_count(p.batch.max_vis_len, tau))
    for inside in (0, 1):
        fb.set_tuning("select_fused", inside)
        try:
            out2, sc2, mass2 = torch.full_like(p.q, 3.0), torch.full_like(sc, -7.0), torch.zeros_like(mass)
            idx, cnt = torch.zeros((p.B, kmax), dtype=torch.int32, device=DEV), torch.zeros((p.B,), dtype=torch.int32, device=DEV)
            fo.focal_attn_score_topk(p.cache, p.batch, p.q, p.scale, tau, out2, sc2, idx, cnt, p.ws(fb.OP_FOCAL_ATTN_SCORE_TOPK, kmax), img_mass=mass2)
        finally:
            fb.set_tuning("select_fused", 0)
        assert torch.equal(out, out2) and torch.equal(sc, sc2) and torch.equal(mass, mass2), f"{what} select_fused {inside}"
        for b, n in enumerate(p.vis_len):
            k = fo.keep_count(n, tau)
            assert int(cnt[b]) == k and np.array_equal(idx[b, :k].cpu().numpy(), oracle.topk(to_np(sc)[b, :n], k)), f"{what} set {b}"
    launches(fb.KERNEL_PARKED_FINISH), launches(fb.KERNEL_ATTN_COMBINE)


# 1, 2, 4 sixteenths of the heads per lane and rounds of them; groups of 1 .. 16; 1 .. 10 kv heads (10, 3 and groups above 8 have no other one-pass form)
@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("Hq,Hkv", [(28, 4), (5, 1), (16, 16), (40, 10), (64, 8), (32, 2), (96, 6), (9, 3)])
def test_edges(Hq, Hkv, d, finish_launches):
    # images of one token less, exactly and one more than a tile, a 64-token block and two; starts that are no multiple of anything
    n = [0, 1, 31, 32, 33, 63, 64, 65, 129, 700, 191]
    case = TinyCase(seed=Hq + d, B=len(n), Hq=Hq, Hkv=Hkv, d=d, n_vis=n, pre=[3, 0, 1, 32, 5, 64, 63, 7, 30, 127, 600],
                    post=[40, 1, 0, 2, 33, 1, 31, 66, 5, 9, 450], dtype="bf16")
    p = problem_from_case(case)
    _check(p, finish_launches, f"{Hq}/{Hkv} d{d}")
    _check(problem_from_case(case, "bshd"), finish_launches, f"{Hq}/{Hkv} d{d} bshd")
    _check(paged_twin(p, 48, 5), finish_launches, f"{Hq}/{Hkv} d{d} paged")


@pytest.mark.parametrize("Hq,Hkv,B,n", [(8, 1, 1, 9000), (4, 1, 1, 2100), (8, 2, 1, 8400), (28, 4, 3, 4097)])      # 72, 18, 67, 21 ranges
def test_many_ranges(Hq, Hkv, B, n, finish_launches):
    case = TinyCase(seed=n, B=B, Hq=Hq, Hkv=Hkv, d=128, n_vis=n, pre=17, post=50, dtype="bf16", spread=1.5)
    _check(problem_from_case(case), finish_launches, f"{Hq}/{Hkv} {n}")


# around the list lengths where a little more than a chip of streams is halved (481, 512 and 513 tokens) and where scoring doubles its ranges
# (7 and 14 of 72 streams, 1 and 2 of 400)
@pytest.mark.parametrize("Hq,Hkv,B,lengths", [(10, 10, 26, (480, 481, 512, 513)), (16, 8, 48, (512, 513)), (8, 8, 9, (7168, 7169)), (10, 10, 40, (1024, 1025))])
def test_ranges_by_size(Hq, Hkv, B, lengths, finish_launches):
    for S in lengths:
        n = [S - 20] + [(S * (b % 7)) // 9 for b in range(1, B)]
        case = TinyCase(seed=S, B=B, Hq=Hq, Hkv=Hkv, d=64 if B > 40 else 128, n_vis=n, pre=11, post=9, dtype="bf16")
        p = problem_from_case(case)
        ref_sc, ref_lse, ref_mass = oracle.focal_score(*p.oracle_args())
        for mode in (1, 0):                                   # parked by its size or not, and always
            fb.set_tuning("score_resident", mode)
            try:
                sc, lse, mass = p.scores(want_lse=True, want_mass=True)
            finally:
                fb.set_tuning("score_resident", 1)
            check_scores(sc, ref_sc, p.vis_len, f"{S} scores")
            assert np.allclose(lse.cpu().numpy(), ref_lse, rtol=2e-5, atol=2e-5) and np.allclose(mass.cpu().numpy(), ref_mass, atol=2e-5)
        out, sc, _, _ = p.focal_attn()
        check_out(out, oracle.decode_attn(*p.oracle_args())[0], f"{S} layer")
        check_scores(sc, ref_sc, p.vis_len, f"{S} layer's scores")


@pytest.mark.parametrize("d", [128, 64])
def test_dead_keys(d, finish_launches):
    """Keys of logit -inf (whole tiles, a whole range, single ones): weight 0, nothing else touched."""
    n, pre, post = [300, 1500], [9, 40], [70, 3]
    case = TinyCase(seed=d, B=2, Hq=16, Hkv=2, d=d, n_vis=n, pre=pre, post=post, dtype="bf16")
    case.q = f32_to_bf16_bits(np.abs(as_f64(case.q)).astype(np.float32) + np.float32(0.25))
    ninf = f32_to_bf16_bits(np.array([-np.inf], np.float32))[0]
    live = [np.ones(s, bool) for s in case.seq_len]
    for b, (lo, hi) in ((0, (0, 64)), (0, (200, 201)), (0, (340, 379)), (1, (64, 224)), (1, (700, 733)), (1, (1542, 1543))):
        live[b][lo:hi] = False
        case.k[b, :, lo:hi, 3] = ninf
    k, v, q = as_f64(case.k), as_f64(case.v), as_f64(case.q)
    sc, lse, out = np.zeros((2, max(n))), np.zeros((2, 16)), np.zeros((2, 16, d))
    for b in range(2):
        for h in range(16):
            lg = k[b, h // 8, : case.seq_len[b]][live[b]] @ q[b, h] * case.scale
            w = np.exp(lg - lg.max())
            lse[b, h] = lg.max() + np.log(w.sum())
            full = np.zeros(case.seq_len[b])
            full[live[b]] = w / w.sum()
            out[b, h] = full @ v[b, h // 8, : case.seq_len[b]]
            sc[b, : n[b]] += full[pre[b]: pre[b] + n[b]] / 16
    _check(problem_from_case(case), finish_launches, f"dead keys d{d}", ref=(sc, lse, sc.sum(1), out))


def test_replayed_from_a_graph_next_to_eager_calls():
    case = TinyCase(seed=3, B=3, Hq=28, Hkv=4, d=128, n_vis=[900, 333, 1200], pre=[5, 0, 64], post=[30, 9, 100], dtype="bf16")
    p = problem_from_case(case)
    kmax = fo.keep_count(1200, 0.05)
    mk = lambda: (torch.zeros_like(p.q), torch.zeros((3, 1200), device=DEV), torch.zeros((3, kmax), dtype=torch.int32, device=DEV),
                  torch.zeros((3,), dtype=torch.int32, device=DEV), torch.empty_like(p.ws(fb.OP_FOCAL_ATTN_SCORE_TOPK, kmax)))
    run = lambda o, s, i, c, ws: fo.focal_attn_score_topk(p.cache, p.batch, p.q, p.scale, 0.05, o, s, i, c, ws)
    for inside in (0, 1):
        fb.set_tuning("select_fused", inside)
        try:
            a, e = mk(), mk()
            run(*a)
            torch.cuda.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g):
                run(*a)
            rng = np.random.default_rng(2)
            for _ in range(4):
                p.q.copy_(torch.from_numpy(rng.standard_normal(p.q.shape).astype(np.float32)).to(DEV).to(torch.bfloat16))
                g.replay()
                run(*e)
                torch.cuda.synchronize()
                assert all(torch.equal(x, y) for x, y in zip(a[:4], e[:4]))
        finally:
            fb.set_tuning("select_fused", 0)


@pytest.mark.parametrize("Hq,Hkv,d", [(28, 4, 128), (64, 8, 64), (5, 1, 128)])
def test_a_batch_of_empty_sequences_alone(Hq, Hkv, d, finish_launches):
    B = 3
    k, v = (torch.randn((B, Hkv, 8, d), device=DEV).to(torch.bfloat16) for _ in range(2))
    p = GpuProblem(k, v, torch.randn((B, Hq, d), device=DEV).to(torch.bfloat16), [0] * B, [0] * B, [0] * B, d ** -0.5)
    assert p.batch.max_seq_len == 0
    for q in (p, paged_twin(p, 4, 1)):
        _, lse, mass = q.scores(want_lse=True, want_mass=True)
        assert (lse == -float("inf")).all() and (mass == 0).all()
        out, _, lse, mass = q.focal_attn(want_lse=True, want_mass=True)
        assert (lse == -float("inf")).all() and (mass == 0).all() and (out == 0).all()
        for inside in (0, 1):
            fb.set_tuning("select_fused", inside)
            try:
                out, mass = torch.full_like(q.q, 3.0), torch.full((B,), 3.0, device=DEV)
                idx, cnt = torch.zeros((B, 1), dtype=torch.int32, device=DEV), torch.full((B,), 3, dtype=torch.int32, device=DEV)
                ws = q.ws(fb.OP_FOCAL_ATTN_SCORE_TOPK, 1)
                fo.focal_attn_score_topk(q.cache, q.batch, q.q, q.scale, 0.1, out, torch.zeros((B, 0), device=DEV), idx, cnt, ws, img_mass=mass)
            finally:
                fb.set_tuning("select_fused", 0)
            assert (cnt == 0).all() and (mass == 0).all() and (out == 0).all()
        assert finish_launches(fb.KERNEL_PARKED_FINISH) > 0


@pytest.mark.parametrize("d", [128, 64])
def test_a_nan_reaches_the_image_mass_of_its_sequence(d):
    """A key that is no number, of the image or of the text: the scores of its sequence are none and so is their sum, the other sequences' stay."""
    case = TinyCase(seed=d, B=4, Hq=16, Hkv=2, d=d, n_vis=[300, 300, 0, 300], pre=[9, 9, 3, 9], post=[70, 70, 50, 70], dtype="bf16")
    clean = problem_from_case(case)
    want_sc, _, want = clean.scores(want_mass=True)
    nan = f32_to_bf16_bits(np.array([np.nan], np.float32))[0]
    case.k[0, 1, 100, 3] = nan                                # image
    case.k[1, 0, 350, 3] = nan                                # text
    case.k[2, 0, 20, 3] = nan                                 # a sequence without an image: a sum of nothing
    p = problem_from_case(case)
    for sc, mass in ((p.scores(want_mass=True)[::2]), (p.focal_attn(want_mass=True)[1::2])):
        assert torch.isnan(sc[:2, :300]).all() and torch.isnan(mass[:2]).all()
        assert mass[2] == 0 and torch.equal(mass[3], want[3]) and torch.equal(sc[3], want_sc[3])


def test_a_process_that_no_longer_trusts_the_exchange_parks_as_before(finish_launches):
    """The parked forms wait for nobody: a call of their size is the same launches after a wave of another form has given up waiting."""
    case = TinyCase(seed=8, B=2, Hq=28, Hkv=4, d=128, n_vis=[900, 400], pre=[5, 0], post=[30, 9], dtype="bf16")
    p = problem_from_case(case)
    kmax = fo.keep_count(900, 0.05)
    results = []
    fb.kernel_timer_enable(fb.KERNEL_TOPK, 8)
    fb.set_tuning("select_fused", 1)
    try:
        for distrust in (0, 1):
            fb.set_tuning("exchange_fallback", distrust)
            sc, idx = torch.zeros((2, 900), device=DEV), torch.zeros((2, kmax), dtype=torch.int32, device=DEV)
            cnt = torch.zeros((2,), dtype=torch.int32, device=DEV)
            fo.focal_score_topk(p.cache, p.batch, p.q, p.scale, 0.05, sc, idx, cnt, p.ws(fb.OP_FOCAL_SCORE_TOPK, kmax))
            assert finish_launches(fb.KERNEL_PARKED_FINISH) == 1 and len(fb.kernel_timer_read(fb.KERNEL_TOPK)) == 0, distrust
            results.append((sc, idx, cnt))
        assert all(torch.equal(a, b) for a, b in zip(*results))
    finally:
        fb.set_tuning("exchange_fallback", 0)
        fb.set_tuning("select_fused", 0)
        fb.kernel_timer_enable(fb.KERNEL_TOPK, 0)


# 7 MiB of logits of 4 x 64 heads are 7168 tokens, 8 MiB 8192
@pytest.mark.parametrize("call,S,parked", [("score", 7168, True), ("score", 7169, False), ("layer", 8192, True), ("layer", 8193, False)])
def test_both_sides_of_the_size_rule(call, S, parked):
    case = TinyCase(seed=S, B=4, Hq=64, Hkv=8, d=64, n_vis=[S - 40, S - 900, 33, 5000], pre=[10, 3, 5, 0], post=[30, 7, 9, 50], dtype="bf16")
    p = problem_from_case(case)
    assert p.batch.max_seq_len == S
    ref_sc, ref_lse, ref_mass = oracle.focal_score(*p.oracle_args())
    kinds = (fb.KERNEL_SCORE_LOGITS, fb.KERNEL_FOCAL_FUSED, fb.KERNEL_PARKED_FINISH, fb.KERNEL_ATTN_COMBINE)
    for k in kinds:
        fb.kernel_timer_enable(k, 16)
    try:
        if call == "score":
            sc, lse, mass = p.scores(want_lse=True, want_mass=True)
            want = (1, 0, int(parked), 0)
        else:
            out, sc, lse, mass = p.focal_attn(want_lse=True, want_mass=True)
            want = (0, 1, int(parked), int(not parked))
        got = tuple(len(fb.kernel_timer_read(k)) for k in kinds)
    finally:
        for k in kinds:
            fb.kernel_timer_enable(k, 0)
    assert got == want or torch.cuda.get_device_properties(0).multi_processor_count != 256, got
    check_scores(sc, ref_sc, p.vis_len, call)
    assert np.allclose(lse.cpu().numpy(), ref_lse, rtol=2e-5, atol=2e-5) and np.allclose(mass.cpu().numpy(), ref_mass, atol=2e-5)
    if call == "layer":
        check_out(out, oracle.decode_attn(*p.oracle_args())[0], "output")
