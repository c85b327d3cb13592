"""Dense attention of lists short enough for one workgroup per stream, and the ranges and merge just above: both sides of each
limit against the oracle, ragged lists among them, the paged cache.  Then the lengths from which half a chip of streams and more is cut."""
import pytest
import torch

import oracle
from paper_2605_17447_amd import binding as fb
from util import TinyCase

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from gpu_util import check_out, paged_twin, problem_from_case


# tiles of 32 tokens that still take one launch, at 256 compute units: by head_dim and streams
@pytest.mark.parametrize("Hq,Hkv,d,B,tiles", [(28, 4, 128, 2, 12), (12, 2, 128, 31, 12), (64, 8, 128, 8, 16), (64, 8, 128, 12, 24),
                                              (28, 4, 128, 32, 32), (14, 2, 64, 3, 8), (64, 8, 64, 16, 24)])
def test_both_sides_of_the_limit(Hq, Hkv, d, B, tiles):
    for extra in (-1, 0, 1):                                   # tokens from the limit: the last is a tile more
        # the longest list decides; the others: short, of one token more than a tile, of nothing but the image
        T = 32 * tiles + extra
        n = [max(T - 50, 1)] + [(7 * b) % 60 if b % 3 else 33 for b in range(1, B)]
        pre, post = [10] + [b % 2 for b in range(1, B)], [T - 10 - n[0]] + [1 + (b % 5) for b in range(1, B)]
        case = TinyCase(seed=tiles + B, B=B, Hq=Hq, Hkv=Hkv, d=d, n_vis=n, pre=pre, post=post, dtype="bf16")
        p = problem_from_case(case)
        assert p.batch.max_seq_len == T
        ref = oracle.decode_attn(*p.oracle_args())[0]
        for q, what in ((p, "bhsd"), (paged_twin(p, 48, 5), "paged")):
            fb.kernel_timer_enable(fb.KERNEL_ATTN_COMBINE, 16)
            try:
                out, _ = q.dense()
                merges = len(fb.kernel_timer_read(fb.KERNEL_ATTN_COMBINE))
            finally:
                fb.kernel_timer_enable(fb.KERNEL_ATTN_COMBINE, 0)
            check_out(out, ref, f"{Hq}/{Hkv} d{d} x{B} {T} {what}")
            assert torch.cuda.get_device_properties(0).multi_processor_count != 256 or merges == int(extra > 0), (T, what, merges)


# streams of 256 compute units, tiles of 32 tokens from which they are cut into three, four or (the last) two ranges
@pytest.mark.parametrize("Hkv,d,B,tiles", [(8, 128, 17, 80), (8, 64, 18, 160), (10, 128, 16, 192), (16, 64, 12, 384), (10, 64, 24, 512)])
def test_streams_that_do_not_fill_the_chip(Hkv, d, B, tiles):
    for T in (32 * tiles - 32, 32 * tiles - 31):
        n = [T - 50] + [(T * (b % 5)) // 16 for b in range(1, B)]
        case = TinyCase(seed=tiles + B, B=B, Hq=Hkv, Hkv=Hkv, d=d, n_vis=n, pre=10, post=40, dtype="bf16")
        p = problem_from_case(case)
        ref, ref_lse = oracle.decode_attn(*p.oracle_args())
        fb.kernel_timer_enable(fb.KERNEL_ATTN_COMBINE, 16)
        try:
            out, lse = p.dense(want_lse=True)
            merges = len(fb.kernel_timer_read(fb.KERNEL_ATTN_COMBINE))
        finally:
            fb.kernel_timer_enable(fb.KERNEL_ATTN_COMBINE, 0)
        check_out(out, ref, f"{Hkv} d{d} x{B} {T}")
        assert torch.allclose(lse.double().cpu(), torch.from_numpy(ref_lse), rtol=2e-5, atol=2e-5)
        assert torch.cuda.get_device_properties(0).multi_processor_count != 256 or merges == int(T > 32 * tiles - 32), (T, merges)
