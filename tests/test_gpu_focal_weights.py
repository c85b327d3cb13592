"""The one-pass layer parks softmax weights relative to the running maximum of their time: logits that rise from tile to tile, that fall,
that jump far up in the wave's last tile, that stay where they are, over one to 32 parked tiles per wave; scores and output against
the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_17447_amd import binding as fb

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from gpu_util import DEV, GpuProblem, check_out, check_scores


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("n", [31, 33, 4000, 32768])
@pytest.mark.parametrize("kind", ["rising", "falling", "jump", "flat"])
def test_maxima_that_move(d, n, kind):
    B, Hq, Hkv, text = 1, 16, 8, 70
    S = n + text
    g = torch.Generator(device=DEV).manual_seed(n + d)
    k, v = (torch.randn((B, Hkv, S, d), generator=g, device=DEV) for _ in range(2))
    q = torch.randn((B, Hq, d), generator=g, device=DEV)
    # the keys' part along the first query of their group, moved over the tokens
    u = q[:, ::2].unsqueeze(2) / q[:, ::2].norm(dim=-1)[:, :, None, None]
    at = torch.linspace(0, 1, S, device=DEV)[None, None, :, None]
    level = {"rising": 3 * at, "falling": 3 - 3 * at, "jump": 4 * (at > 1 - 20 / S).float(), "flat": 0 * at}[kind]
    if kind == "flat":
        k = k * 0 + u
    p = GpuProblem((k + level * u).bfloat16(), v.bfloat16(), q.bfloat16(), [S], [text // 2], [n], d ** -0.5)
    ref_sc, _, _ = oracle.focal_score(*p.oracle_args())
    want, _ = oracle.decode_attn(*p.oracle_args())
    fb.set_tuning("focal_fused", 2)
    try:
        out, sc, _, _ = p.focal_attn()
    finally:
        fb.set_tuning("focal_fused", 1)
    check_scores(sc, ref_sc, p.vis_len, f"{kind} {n}")
    check_out(out, want, f"{kind} {n}")
