"""Dense and pruned attention of bf16 caches with runs of keys whose logits are -inf, whole first tiles of a wave among them: weight 0, the other
keys' weights untouched, in every way a workgroup's result leaves the kernel."""
import numpy as np
import pytest
import torch

from paper_2605_17447_amd import binding as fb
from util import TinyCase, as_f64, f32_to_bf16_bits

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from gpu_util import DEV, check_out, paged_twin, problem_from_case


def _reference(case, use):
    """Softmax in 64 bits over the positions use[b]."""
    k, v, q = as_f64(case.k), as_f64(case.v), as_f64(case.q)
    G, out, lse = case.Hq // case.Hkv, np.zeros((case.B, case.Hq, case.d)), np.zeros((case.B, case.Hq))
    for b in range(case.B):
        for h in range(case.Hq):
            lg = k[b, h // G, use[b]] @ q[b, h] * case.scale
            w = np.exp(lg - lg.max())
            out[b, h] = w @ v[b, h // G, use[b]] / w.sum()
            lse[b, h] = lg.max() + np.log(w.sum())
    return out, lse


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("fill", [-np.inf, -3.0e38])
@pytest.mark.parametrize("B,n,post", [(2, 200, 40), (2, 900, 300), (1, 5000, 40)])      # one workgroup per stream; ranges and their merge
def test_dead_tiles(B, n, post, fill, d):
    case = TinyCase(seed=n + d, B=B, Hq=8, Hkv=2, d=d, n_vis=n, pre=16, post=post, dtype="bf16")
    case.q = f32_to_bf16_bits(np.abs(as_f64(case.q)).astype(np.float32) + np.float32(1.0))
    S = int(case.seq_len[0])
    dead = np.zeros(S, bool)
    for lo, hi in ((0, 8), (16, 150), (170, 171), (S // 2, S // 2 + 100), (S - 33, S - 1)):
        dead[lo:hi] = True
    # every component: a finite fill gives logits far below any live one, or -inf
    bits = f32_to_bf16_bits(np.array([fill], np.float32))[0]
    case.k[:, :, dead] = bits
    live = [np.nonzero(~dead)[0]] * B
    ref, ref_lse = _reference(case, live)
    p = problem_from_case(case)
    kmax = n // 2
    idx = torch.arange(0, 2 * kmax, 2, dtype=torch.int32, device=DEV).repeat(B, 1).contiguous()
    cnt = torch.full((B,), kmax, dtype=torch.int32, device=DEV)
    kept = np.concatenate([np.arange(16), 16 + np.arange(0, 2 * kmax, 2), np.arange(16 + n, S)])
    ref_s, _ = _reference(case, [kept[~dead[kept]]] * B)
    for x, what in ((p, "bhsd"), (paged_twin(p, 48, 3), "paged")):
        for waves in (4, 8):
            fb.set_tuning("attn_waves", waves)
            out, lse = x.dense(want_lse=True)
            fb.set_tuning("attn_waves", 4)
            check_out(out, ref, f"dense {what}, {waves} waves")
            assert np.allclose(lse.cpu().numpy(), ref_lse, rtol=2e-5, atol=2e-5)
        for merge, splits in ((1, 0), (1, 1), (1, 3), (0, 3)):
            fb.set_tuning("attn_merge", merge)
            fb.set_tuning("splits_sparse", splits)
            try:
                check_out(x.sparse(idx, cnt), ref_s, f"pruned {what}, merge {merge}, ranges {splits}")
            finally:
                fb.set_tuning("attn_merge", 1)
                fb.set_tuning("splits_sparse", 0)
