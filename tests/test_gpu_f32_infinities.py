"""fp32 caches whose logits leave fp32's range: a key of logit -inf has weight 0, and so has a run of keys below the
type's lowest value as long as any other key is above it; infinities do not spread to the other keys' weights."""
import numpy as np
import pytest
import torch

import paper_2605_17447_amd as fo
from util import TinyCase

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from gpu_util import DEV, check_out, check_scores, problem_from_case

LOWEST = float(np.finfo(np.float32).min)


def _reference(case, use):
    """Softmax over the positions `use[b]` in 64 bits: outputs [B, Hq, d], head-averaged weights [B, S]."""
    G = case.Hq // case.Hkv
    out = np.zeros((case.B, case.Hq, case.d))
    mean = np.zeros((case.B, case.S))
    for b in range(case.B):
        for h in range(case.Hq):
            k, v = case.k[b, h // G].astype(np.float64)[use[b]], case.v[b, h // G].astype(np.float64)[use[b]]
            lg = k @ case.q[b, h].astype(np.float64) * case.scale
            w = np.exp(lg - lg.max())
            w /= w.sum()
            out[b, h] = w @ v
            mean[b, use[b]] += w / case.Hq
    return out, mean


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("kind", ["one key of -inf", "runs of -inf", "runs below the lowest value"])
def test_keys_out_of_range(kind, d):
    n_vis, pre, post = [60, 900], [7, 20], [9, 70]
    case = TinyCase(seed=31 + d, B=2, Hq=8, Hkv=2, d=d, n_vis=n_vis, pre=pre, post=post, dtype="f32")
    case.q = np.abs(case.q) + np.float32(0.5)                # a key of one huge component has logits of one sign
    rows = [np.zeros(s, bool) for s in case.seq_len]
    if kind == "one key of -inf":
        rows[0][5] = rows[1][500] = True
        fill = -np.inf
    else:                                                    # a whole tile of the first wave, of later ones, the last rows
        for lo, hi in ((0, 16), (40, 64), (320, 420), (980, 990)):
            for r in rows:
                r[lo:hi] = True
        fill = -np.inf if kind == "runs of -inf" else LOWEST
    for b, r in enumerate(rows):
        if fill == LOWEST:
            case.k[b, :, : len(r)][:, r] = LOWEST            # every component: logits of about -1e40
        else:
            case.k[b, :, : len(r)][:, r, 3] = fill
    p = problem_from_case(case)
    every = [np.arange(s) for s in case.seq_len]
    want, mean = _reference(case, every)
    image = np.zeros((case.B, max(n_vis)))
    for b in range(case.B):
        image[b, : n_vis[b]] = mean[b, pre[b]: pre[b] + n_vis[b]]
    check_out(p.dense()[0], want, f"{kind} dense")
    sc, lse, mass = p.scores(want_lse=True, want_mass=True)
    check_scores(sc, image, n_vis, f"{kind} scores")
    assert torch.isfinite(lse).all() and np.abs(mass.cpu().numpy() - image.sum(1)).max() <= 1e-5
    out, sc, _, mass = p.focal_attn(want_mass=True)
    check_out(out, want, f"{kind} focal layer")
    check_scores(sc, image, n_vis, f"{kind} focal layer's scores")
    assert np.abs(mass.cpu().numpy() - image.sum(1)).max() <= 1e-5
    # pruned: every second image token, masked ones among them
    kmax = max(n_vis) // 2
    idx, cnt = torch.zeros((case.B, kmax), dtype=torch.int32), torch.zeros(case.B, dtype=torch.int32)
    use = []
    for b, n in enumerate(n_vis):
        idx[b, : n // 2] = torch.arange(0, n // 2 * 2, 2, dtype=torch.int32)
        cnt[b] = n // 2
        pos = np.arange(case.seq_len[b])
        use.append(np.concatenate([pos[: pre[b]], pre[b] + np.arange(0, n // 2 * 2, 2), pos[pre[b] + n:]]))
    check_out(p.sparse(idx.to(DEV), cnt.to(DEV)), _reference(case, use)[0], f"{kind} pruned")


@pytest.mark.parametrize("d", [128, 64])
def test_a_nan_stays_in_its_kv_head(d):
    # the plain kernels' behaviour: the sums of the heads that see a NaN are no numbers (their outputs are zero rows), the others' are untouched
    case = TinyCase(seed=41, B=2, Hq=8, Hkv=2, d=d, n_vis=[60, 900], pre=[7, 20], post=[9, 70], dtype="f32")
    clean = problem_from_case(case).dense()[0]
    case.k[1, 1, 333, 2] = np.nan
    p = problem_from_case(case)
    out = p.dense()[0]
    assert torch.equal(out[0], clean[0]) and torch.equal(out[1, :4], clean[1, :4])
    assert (out[1, 4:] == 0).all()
    sc = p.scores()[0]
    assert torch.isfinite(sc[0, :60]).all() and torch.isnan(sc[1, :900]).all()
