"""The register-resident kernels deal their workgroups over unlike sequences from a table that every wave works out: batches of one to
four rounds of 64 sequences, lengths of one token next to the longest, text-heavy sequences, all but one alike.  Against the forms that
need no table, which share no code with it."""
import numpy as np
import pytest
import torch

from paper_2605_17447_amd import binding as fb

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from gpu_util import DEV, GpuProblem


def _lengths(rng, B, kind):
    n, text = np.full(B, 1500), np.full(B, 40)
    if kind == "spread":
        n = rng.integers(0, 1500, B)
    elif kind == "one":                     # all alike but the last
        n[-1] = 37
    elif kind == "short":                   # one long, the others a few tokens
        n[1:], text[1:] = 1, rng.integers(0, 2, B - 1)
    elif kind == "text":
        n, text = rng.integers(1, 100, B), rng.integers(1, 1400, B)
    n[0] = 1500
    return n, text


@pytest.mark.parametrize("B,Hq,Hkv,d", [(2, 14, 2, 64), (63, 8, 1, 128), (64, 28, 4, 128), (65, 16, 2, 64), (130, 16, 2, 128), (200, 4, 1, 64)])
@pytest.mark.parametrize("kind", ["spread", "one", "short", "text"])
def test_ragged_batches_of_one_to_four_rounds(B, Hq, Hkv, d, kind):
    rng = np.random.default_rng(B)
    n, text = _lengths(rng, B, kind)
    S = int((n + text).max())
    g = torch.Generator(device=DEV).manual_seed(B)
    k, v = (torch.randn((B, Hkv, S, d), generator=g, device=DEV).bfloat16() for _ in range(2))
    q = torch.randn((B, Hq, d), generator=g, device=DEV).bfloat16()
    p = GpuProblem(k, v, q, n + text, text // 2, n, d ** -0.5)
    got = {}
    for mode in (2, 0):
        fb.set_tuning("score_resident", mode)
        fb.set_tuning("focal_fused", mode)
        try:
            sc, lse, mass = p.scores(True, True)
            out, sc2, lse2, mass2 = p.focal_attn(True, True)
        finally:
            fb.set_tuning("score_resident", 1)
            fb.set_tuning("focal_fused", 1)
        got[mode] = [x.float().cpu().numpy() for x in (sc, sc2, lse, lse2, mass, mass2, out)]
    for a, b, what in zip(got[2], got[0], ("scores", "layer's scores", "lse", "layer's lse", "mass", "layer's mass", "out")):
        if what == "out":
            # two bf16 forms, each within 2e-2 of its row's maximum of the truth
            assert (np.abs(a - b).max(-1) <= 4e-2 * np.abs(b).max(-1)).all(), what
        elif "lse" in what:
            assert np.allclose(a, b, rtol=0, atol=2e-5), what
        else:
            # each within 1e-6 of the truth; the mass is a sum of up to 1500 scores, at most 1
            assert np.abs(a - b).max() <= (2e-6 if "scores" in what else 1e-5), (what, np.abs(a - b).max())
