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


@pytest.mark.parametrize("dtype,d,splits", [("bf16", 128, 1), ("bf16", 64, 3), ("bf16", 128, 4), ("f32", 128, 1), ("f32", 64, 2)])
def test_rows_outside_the_set_are_never_read(dtype, d, splits):
    """No text, sets that end inside a tile, junk entries behind them that name rows of NaN: nothing of those may reach the output."""
    n = [500, 77, 40, 1]
    case = TinyCase(seed=52 + splits, B=4, Hq=6, Hkv=2, d=d, n_vis=n, pre=[0] * 4, post=[0] * 4, dtype=dtype)
    p = problem_from_case(case)
    rng = np.random.default_rng(d + splits)
    kmax, cnt = 500, np.array([301, 33, 17, 1], np.int32)
    idx = np.zeros((4, kmax), np.int32)
    for b in range(4):
        idx[b, : cnt[b]] = np.sort(rng.permutation(n[b])[: cnt[b]])
    want, _ = oracle.decode_attn(*p.oracle_args(), idx, cnt)
    for b in range(4):
        others = np.setdiff1d(np.arange(n[b]), idx[b, : cnt[b]])
        if others.size:
            idx[b, cnt[b]:] = rng.choice(others, kmax - cnt[b])
            p.cache.k[b, :, torch.from_numpy(others).to(DEV)] = float("nan")
            p.cache.v[b, :, torch.from_numpy(others).to(DEV)] = float("nan")
    try:
        fb.set_tuning("splits_sparse", splits)
        check_out(p.sparse(torch.from_numpy(idx).to(DEV), torch.from_numpy(cnt).to(DEV)), want, f"{dtype} d={d} splits={splits}")
    finally:
        fb.set_tuning("splits_sparse", 0)


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("paged", [False, True])
def test_fp32_tiles_in_turn(d, paged):
    """Lists of fewer tiles than waves, of one to four tiles per wave with a remainder, and of nothing."""
    n, pre, post = [0, 5, 900, 300, 60], [0, 3, 40, 16, 17], [0, 0, 61, 1, 500]
    case = TinyCase(seed=61, B=5, Hq=6, Hkv=2, d=d, n_vis=n, pre=pre, post=post, dtype="f32")
    p = problem_from_case(case)
    if paged:
        p = paged_twin(p, 16, 5)
    rng = np.random.default_rng(d)
    kmax, cnt = 300, np.array([0, 1, 300, 16, 60], np.int32)
    idx = np.zeros((5, kmax), np.int32)
    for b in range(5):
        idx[b, : cnt[b]] = np.sort(rng.permutation(n[b])[: cnt[b]])
    want, _ = oracle.decode_attn(*p.oracle_args(), idx, cnt)
    junk = np.where(np.arange(kmax)[None] < cnt[:, None], idx, rng.choice([-1, 2 ** 31 - 1], (5, kmax))).astype(np.int32)
    try:
        for splits in (1, 2, 5):
            fb.set_tuning("splits_sparse", splits)
            check_out(p.sparse(torch.from_numpy(junk).to(DEV), torch.from_numpy(cnt).to(DEV)), want, f"d={d} paged={paged} splits={splits}")
    finally:
        fb.set_tuning("splits_sparse", 0)
