"""Pruned attention of bf16 caches asks for the set's entries before it knows any length, and deals short lists to its waves in turn:
sets far below kmax with junk behind them, empty sets, sequences without text or of a single token.  A call whose ranges merge
inside the launch and one without an exchange slot give the same bits."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_17447_amd import binding as fb
from util import TinyCase

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from gpu_util import DEV, check_out, paged_twin, problem_from_case


@pytest.mark.parametrize("d,splits", [(128, 1), (128, 2), (128, 4), (64, 1), (64, 3)])
@pytest.mark.parametrize("paged", [False, True])
def test_short_sets_with_junk_behind_them(d, splits, paged):
    case = TinyCase(seed=41 + splits, B=6, Hq=6, Hkv=2, d=d, n_vis=[700, 700, 1, 300, 0, 900], pre=[40, 0, 0, 33, 5, 300],
                    post=[90, 0, 0, 31, 27, 700], dtype="bf16")
    p = problem_from_case(case)
    if paged:
        p = paged_twin(p, 16, 3)
    rng = np.random.default_rng(d + splits)
    kmax, cnt = 700, np.array([1, 64, 1, 0, 0, 513], np.int32)
    idx = np.zeros((6, kmax), np.int32)
    for b, n in enumerate(p.vis_len):
        idx[b, : cnt[b]] = np.sort(rng.permutation(n)[: cnt[b]])
    want, _ = oracle.decode_attn(*p.oracle_args(), idx, cnt)
    junk = np.where(np.arange(kmax)[None] < cnt[:, None], idx, rng.choice([-1, 0, 2 ** 31 - 1, -2 ** 31], (6, kmax))).astype(np.int32)
    got = []
    try:
        fb.set_tuning("splits_sparse", splits)
        for distrust in (0, 1):
            fb.set_tuning("exchange_fallback", distrust)
            got.append(p.sparse(torch.from_numpy(junk).to(DEV), torch.from_numpy(cnt).to(DEV)).clone())
            check_out(got[-1], want, f"d={d} splits={splits} paged={paged} distrust={distrust}")
    finally:
        fb.set_tuning("splits_sparse", 0)
        fb.set_tuning("exchange_fallback", 0)
    assert torch.equal(got[0], got[1])
