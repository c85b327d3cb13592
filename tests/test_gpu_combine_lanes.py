"""The merge of output partials at the edges of its forms: maxima walked by every thread up to 12 partials, one per lane up to 32, a
reduction through LDS beyond; sequences of which most ranges are empty, and partials whose maxima lie far apart."""
import pytest
import torch

import oracle
from paper_2605_17447_amd import binding as fb
from util import TinyCase, as_f64, store

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from gpu_util import check_out, problem_from_case


@pytest.mark.parametrize("splits", [2, 12, 13, 31, 32, 33])
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 128)])
def test_partials_at_the_edges(splits, dtype, d):
    n = [4300, 40, 1, 2000]
    case = TinyCase(seed=81 + splits, B=4, Hq=6, Hkv=2, d=d, n_vis=n, pre=[3, 0, 0, 50], post=[10, 1, 0, 0], dtype=dtype)
    k = as_f64(case.k)
    k[0, :, 4000:] *= 6.0                           # one range's logits far above all others
    case.k = store(k, dtype)
    p = problem_from_case(case)
    want, _ = oracle.decode_attn(*p.oracle_args())
    try:
        fb.set_tuning("splits_dense", splits)
        check_out(p.dense()[0], want, f"{dtype} d={d} splits={splits}")
    finally:
        fb.set_tuning("splits_dense", 0)
