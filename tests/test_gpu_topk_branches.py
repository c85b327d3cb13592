"""Branches of the register select: waves with and without a score that has a sign bit, image spans that end inside a wave, and
thresholds whose equal keys are all, partly or one by one in the set."""
import numpy as np
import pytest

from test_gpu_topk import assert_same, expect, run_topk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,W", [(63, 64), (64, 64), (255, 4096), (257, 4096), (4095, 4096), (4097, 8192), (8191, 8192), (8193, 16384), (16383, 16384)])
@pytest.mark.parametrize("tau", [0.02, 0.5])
def test_signs_in_one_wave_and_shared_thresholds(n, W, tau):
    rng = np.random.default_rng(n)
    k = max(1, int(np.ceil(tau * n - 1e-9)))
    rows = []
    for kind in range(6):
        s = rng.random(W).astype(np.float32)
        order = np.argsort(-s[:n], kind="stable")
        if kind == 1:                        # a sign bit at one place only, on a zero or a number
            s[rng.integers(n)] = -0.0
            s[rng.integers(n)] = -1.0
        elif kind == 2:                      # the keys equal to the threshold are exactly those wanted
            s[order[max(0, k - 3): k]] = s[order[k - 1]]
        elif kind == 3:                      # some of them are not wanted
            s[order[max(0, k - 3): k + 5]] = s[order[k - 1]]
        elif kind == 4:                      # all keys equal: no window to search
            s[:] = 0.25
        elif kind == 5:                      # zeros of both signs on the threshold
            s[order[max(0, k - 2):]] = 0.0
            s[order[max(0, k - 2)::2]] = -0.0
        s[n:] = -np.inf if kind == 1 else np.inf          # past the span: never looked at
        rows.append(s)
    scores = np.stack(rows)
    idx, cnt = run_topk(scores, [n] * 6, tau)
    assert_same(idx, cnt, expect(scores, [n] * 6, tau), f"n={n}")
