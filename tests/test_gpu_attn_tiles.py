"""Dense and pruned attention on the matrix cores for every short tile count per wave: the pipelined loop leaves one or
two tiles, row look-ups come in pairs of tiles, the last tile may hold a single row."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_17447_amd import binding as fb
from util import TinyCase

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from gpu_util import DEV, check_out, paged_twin, problem_from_case


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("tiles", [1, 2, 3, 4, 5, 6])
def test_tiles_per_wave(tiles, d):
    """nsplit 1: eight waves share the list, so 256 * tiles positions give every wave `tiles` tiles."""
    lens = [256 * tiles, 256 * tiles - 31, 256 * (tiles - 1) + 1]
    case = TinyCase(seed=70 + tiles, B=3, Hq=6, Hkv=2, d=d, n_vis=[n // 2 for n in lens], pre=[n // 4 for n in lens],
                    post=[n - n // 2 - n // 4 for n in lens], dtype="bf16")
    for layout, paged in (("bhsd", False), ("bshd", False), ("bhsd", True)):
        p = problem_from_case(case, layout)
        if paged:
            p = paged_twin(p, 16, tiles)
        oc = p.oracle_args()
        rng = np.random.default_rng(tiles)
        kmax = max(p.vis_len)
        idx, cnt = np.zeros((3, kmax), np.int32), np.zeros(3, np.int32)
        for b, n in enumerate(p.vis_len):
            k = n if b == 0 else max(1, n - 3) if n else 0            # (sequence 0: every position, 256 * tiles of them)
            idx[b, :k] = np.sort(rng.permutation(n)[:k])
            cnt[b] = k
        dense, _ = oracle.decode_attn(*oc)
        sparse, _ = oracle.decode_attn(*oc, idx, cnt)
        try:
            for nsplit in (1, 2):
                for key in ("splits_dense", "splits_sparse"):
                    fb.set_tuning(key, nsplit)
                check_out(p.dense()[0], dense, f"dense d={d} tiles={tiles} {layout} paged={paged} nsplit={nsplit}")
                check_out(p.sparse(torch.from_numpy(idx).to(DEV), torch.from_numpy(cnt).to(DEV)), sparse,
                          f"sparse d={d} tiles={tiles} {layout} paged={paged} nsplit={nsplit}")
        finally:
            for key in ("splits_dense", "splits_sparse"):
                fb.set_tuning(key, 0)
