"""Workspace sizes (host only): a size asked for once, for the longest sequences of a run, serves every shorter one, and
one asked for a full batch serves the layers' calls on fewer sequences wherever the kernels' own choices allow it."""
import ctypes

import pytest

from paper_2605_17447_amd import binding as fb
from test_abi_host import FAKE, _bv, _kv

HEADS = [(28, 4), (64, 8), (32, 8), (16, 2), (8, 1), (4, 1), (16, 1), (5, 5)]
OPS = {"score": fb.OP_FOCAL_SCORE, "dense": fb.OP_DENSE_DECODE_ATTN, "sparse": fb.OP_SPARSE_DECODE_ATTN,
       "focal": fb.OP_FOCAL_ATTN_SCORE, "focal_topk": fb.OP_FOCAL_ATTN_SCORE_TOPK}


@pytest.fixture(scope="module")
def need():
    lib = fb.load_library()

    def size(op, dtype, d, heads, B, S, N, kmax=0):
        kv, bv = _kv(dtype, Hkv=heads[1], d=d, S=S), _bv(B, S, N)
        n = lib.fastocr_workspace_bytes(OPS[op], ctypes.byref(kv), ctypes.byref(bv), heads[0], kmax)
        assert n > 0
        return n

    return size


def _never_shrinks(sizes):
    top = 0
    for what, n in sizes:
        assert n >= top, f"{what}: {n} bytes, a smaller problem needs {top}"
        top = n


@pytest.mark.parametrize("dtype,d", [(fb.BF16, 128), (fb.BF16, 64), (fb.F32, 128), (fb.F32, 64), (fb.BF16, 96)])
@pytest.mark.parametrize("op", list(OPS))
def test_a_size_never_shrinks_as_sequences_grow(need, op, dtype, d):
    images = list(range(1, 2100, 31)) + [2080, 2081] + list(range(2100, 33000, 493)) + [16351, 16384, 16412]
    for heads in HEADS:
        for B in (1, 4, 12, 100):
            _never_shrinks((f"{heads} batch {B}, {n} image tokens", need(op, dtype, d, heads, B, n + 200, n, 0))
                           for n in sorted(images))
            _never_shrinks((f"{heads} batch {B}, {t} text tokens", need(op, dtype, d, heads, B, 300 + t, 300, 0))
                           for t in range(0, 4000, 61))


def test_pruned_attention_sizes_around_the_range_counts(need):
    # the automatic number of ranges of a list falls from four to three after 32 tiles of 32 tokens: a size for the longer list covers it
    for d in (128, 64):
        for heads in ((28, 4), (12, 2), (8, 1)):
            for B in (1, 2, 8, 16, 64):
                _never_shrinks((f"{heads} batch {B}, {tiles} tiles", need("sparse", fb.BF16, d, heads, B, 20000, 19000, 32 * tiles - 1000))
                               for tiles in range(32, 80))


def test_a_size_for_a_batch_covers_fewer_sequences(need):
    for heads in HEADS:
        for d in (128, 64):
            for n in (33, 100, 300, 1000, 5000):
                for op in ("dense", "sparse"):
                    _never_shrinks((f"{op} fp32 {heads} d={d} batch {B}, {n} image tokens", need(op, fb.F32, d, heads, B, n + 60, n, 500))
                                   for B in range(1, 700, 3))
                if heads != (5, 5):
                    _never_shrinks((f"focal bf16 {heads} d={d} batch {B}, {n} image tokens", need("focal", fb.BF16, d, heads, B, n + 60, n))
                                   for B in range(1, 256, 5))


@pytest.mark.parametrize("op", list(OPS))
def test_a_bf16_size_for_a_batch_covers_fewer_sequences(need, op):
    batches = list(range(1, 140)) + [160, 192, 255, 256, 257, 300, 511, 512, 513, 900]
    for heads in HEADS:
        for d in (128, 64):
            for n in (33, 150, 300, 1000, 5000, 17000):
                _never_shrinks((f"{op} {heads} d={d} batch {B}, {n} tokens", need(op, fb.BF16, d, heads, B, n, n - 20, 500)) for B in batches)


@pytest.mark.parametrize("d", [128, 64])
def test_the_static_scratch_serves_every_bf16_group_size(d):
    # dense attention of up to a chip of streams (256 compute units, 16 heads a group), or more of single ranges that fit
    lib = fb.load_library()
    for G in (1, 2, 5, 7, 8, 16):
        for Hkv in (1, 2, 4, 8, 16):
            for B in (1, 2, 3, 7, 16, 17, 23, 40, 100, 250):
                if G * Hkv > 256 or B * G * Hkv > 16000:
                    continue
                for S in (64, 500, 1000, 4000, 20000):
                    kv, bv = _kv(fb.BF16, Hkv=Hkv, d=d, S=S), _bv(B, S, S // 2)
                    n = lib.fastocr_workspace_bytes(fb.OP_DENSE_DECODE_ATTN, ctypes.byref(kv), ctypes.byref(bv), G * Hkv, 0)
                    assert 0 < n <= fb.STATIC_SCRATCH_BYTES, (G, Hkv, B, S, n)


def test_the_static_scratch_serves_every_fp32_group_size():
    # fp32 caches leave at most two ranges per compute unit and query head of a group, 16 heads: 4.3 MB at head_dim 128
    lib = fb.load_library()
    for G in range(1, 17):
        for Hkv in (1, 2, 4, 8, 16):
            if G * Hkv > 256:
                continue
            for d in (64, 128):
                for B in (1, 2, 3, 7, 16, 40, 100, 250):
                    if B * G * Hkv > 16000:                  # more rows than the buffer holds at one range each
                        continue
                    for S in (64, 1000, 20000):
                        kv, bv = _kv(fb.F32, Hkv=Hkv, d=d, S=S), _bv(B, S, S // 2)
                        n = lib.fastocr_workspace_bytes(fb.OP_DENSE_DECODE_ATTN, ctypes.byref(kv), ctypes.byref(bv), G * Hkv, 0)
                        assert 0 < n <= fb.STATIC_SCRATCH_BYTES, (G, Hkv, d, B, S, n)
