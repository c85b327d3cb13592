"""Layers enqueued together never have an output where another of them reads or writes: the overlap test itself (csrc/apart.hpp, compiled
here) against every pair of spans, and outputs in the pool of a paged cache, which only the binding can see."""
import ctypes
import os
import random
import subprocess
import types

import pytest
import torch

from paper_2605_17447_amd import _build
from paper_2605_17447_amd import binding as fb

SHIM = r"""
#include "apart.hpp"
using namespace fastocr;
// spans as (lo, hi) pairs; reads have the layer that owns them (-1: nobody).  0: outputs overlap, 1: an output lies in a read span, 2: apart
extern "C" int look(int n, const uint64_t *out, int m, const uint64_t *read, const int *own)
{
    Outputs<32> o;
    Span s[32];
    for (int i = 0; i < n; ++i) s[i] = span_of((const void *)out[2 * i], (int64_t)(out[2 * i + 1] - out[2 * i]));
    if (!o.set(s, n)) return 0;
    for (int i = 0; i < m; ++i)
        if (!o.apart(span_of((const void *)read[2 * i], (int64_t)(read[2 * i + 1] - read[2 * i])), own[i])) return 1;
    return 2;
}
"""


@pytest.fixture(scope="module")
def look(tmp_path_factory):
    d = tmp_path_factory.mktemp("apart")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-I", _build.CSRC, str(d / "shim.cpp"), "-o", str(d / "shim.so")])
    f = ctypes.CDLL(str(d / "shim.so")).look

    def run(outs, reads):
        flat = lambda xs: (ctypes.c_uint64 * max(1, 2 * len(xs)))(*(v for lo, hi in xs for v in (lo, hi)))      # noqa: E731
        return f(len(outs), flat(outs), len(reads), flat([r for r, _ in reads]), (ctypes.c_int * max(1, len(reads)))(*(o for _, o in reads)))
    return run


@pytest.mark.parametrize("seed", range(4))
def test_the_overlap_test_against_all_pairs(look, seed):
    rng, seen = random.Random(seed), set()
    for _ in range(3000):
        n, space = rng.randint(2, 32), rng.choice([200, 2000, 40000])
        size = rng.randint(1, 12)                                        # the layers' outputs are of one size
        outs = [(lo, lo + size) for lo in (rng.randint(1, space) for _ in range(n))]
        if rng.random() < 0.8:                                           # apart, in any order, often neighbours without a gap
            at, outs = 1, []
            for _ in range(n):
                at += rng.choice([0, 0, rng.randint(0, max(1, space // n))])
                outs.append((at, at + size))
                at += size
            rng.shuffle(outs)
        reads = [((lo, lo + rng.randint(0, 40)), rng.choice([-1, rng.randrange(n)])) for lo in (rng.randint(1, space) for _ in range(rng.randint(0, 6)))]
        meet = lambda a, b: max(a[0], b[0]) < min(a[1], b[1])            # noqa: E731
        want = 2
        if any(meet(outs[i], outs[j]) for i in range(n) for j in range(i)):
            want = 0
        elif any(meet(o, r) for r, own in reads for i, o in enumerate(outs) if i != own):
            want = 1
        assert look(outs, reads) == want, (outs, reads)
        seen.add(want)
    assert seen == {0, 1, 2}


@pytest.fixture
def recorded(monkeypatch):
    """The names of the entry points that a call reaches, native or through ctypes; nothing runs."""
    if fb._raw_stream is None:
        pytest.skip("this torch has no stream handles to pass on")
    real, seen = fb.load_library(), []
    proto = lambda name: (lambda *a: seen.append(name) or 0)             # noqa: E731
    P, I, I64, F, SZ, KV, BV = (ctypes.c_void_p, ctypes.c_int, ctypes.c_int64, ctypes.c_float, ctypes.c_size_t, ctypes.POINTER(fb.KvView),
                                ctypes.POINTER(fb.BatchView))
    one = ctypes.CFUNCTYPE(I, KV, BV, P, I, F, P, P, I64, P, P, SZ, P)(proto("one"))
    layers = ctypes.CFUNCTYPE(I, I, KV, BV, P, I, F, P, P, I64, P, P, SZ, P)(proto("layers"))
    at = lambda f: ctypes.cast(f, P).value                               # noqa: E731
    assert fb._call is not None
    fb._call.bind(fb.KvCache, fb.SeqBatch, lambda: 0, lambda dev: 0x5000, lambda: True, *([at(one)] * 7))
    fb._call.bind_layers(at(layers))
    monkeypatch.setattr(fb, "_lib", types.SimpleNamespace(fastocr_sparse_decode_attn=one, fastocr_sparse_decode_attn_layers=layers))
    monkeypatch.setattr(fb, "_stream_handle", lambda s: None)
    yield seen, fb._call
    monkeypatch.undo()
    fb._bind_call(real)


@pytest.mark.parametrize("native", [True, False])
@pytest.mark.parametrize("where,goes", [("apart", ["layers"]), ("right behind a pool", ["layers"]), ("a page of another layer", ["one"] * 3),
                                        ("a page of its own", ["one"] * 3), ("the last page", ["one"] * 3), ("v", ["one"] * 3)])
def test_an_output_in_the_pool_of_a_paged_cache(recorded, monkeypatch, native, where, goes):
    seen, call = recorded
    B, H, d, page, pages = 2, 2, 64, 16, 6
    pool = page * H * d * pages
    mem = torch.zeros(8 * pool + 64, dtype=torch.bfloat16)               # six pools with room behind each
    pools = [mem[i * (pool + B * H * d):][:pool].view(pages, H, page, d) for i in range(6)]
    caches = [fb.KvCache(pools[2 * l], pools[2 * l + 1], block_table=torch.zeros(B, 3, dtype=torch.int32)) for l in range(3)]
    i32 = lambda *s: torch.zeros(*s, dtype=torch.int32)                  # noqa: E731
    batch = fb.SeqBatch(i32(B), i32(B), i32(B), 40, 20)
    qs = [torch.zeros(B, H, d, dtype=torch.bfloat16) for _ in range(3)]
    outs = [torch.zeros_like(q) for q in qs]
    size = B * H * d
    behind = lambda i: mem[i * (pool + size) + pool:][:size].view(B, H, d)                 # noqa: E731
    within = lambda t, off: t.view(-1)[off:off + size].view(B, H, d)                       # noqa: E731
    if where == "right behind a pool":
        outs[0], outs[2] = behind(2), behind(4)
    elif where == "a page of another layer":
        outs[0] = within(pools[4], 128)
    elif where == "a page of its own":
        outs[1] = within(pools[2], 128)
    elif where == "the last page":
        outs[2] = mem[pool - 1:][:size].view(B, H, d)                    # one element of it
    elif where == "v":
        outs[0] = within(pools[5], 0)
    if not native:
        monkeypatch.setattr(fb, "_call", None)
    else:
        monkeypatch.setattr(fb, "_call", call)
    fb.sparse_decode_attn_layers(caches, batch, qs, 0.125, i32(B, 4), i32(B), outs, torch.zeros(256, dtype=torch.uint8))
    assert seen == goes


@pytest.mark.parametrize("native", [True, False])
def test_layers_of_unlike_query_heads_go_one_by_one(recorded, monkeypatch, native):
    seen, call = recorded
    monkeypatch.setattr(fb, "_call", call if native else None)
    i32 = lambda *s: torch.zeros(*s, dtype=torch.int32)                  # noqa: E731
    caches = [fb.KvCache(*(torch.zeros(2, 2, 40, 64, dtype=torch.bfloat16) for _ in range(2))) for _ in range(3)]
    qs = [torch.zeros(2, h, 64, dtype=torch.bfloat16) for h in (4, 8, 4)]
    fb.sparse_decode_attn_layers(caches, fb.SeqBatch(i32(2), i32(2), i32(2), 40, 20), qs, 0.125, i32(2, 4), i32(2), [torch.zeros_like(q) for q in qs],
                                 torch.zeros(256, dtype=torch.uint8))
    assert seen == ["one"] * 3
