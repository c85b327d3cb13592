"""Layers enqueued together whose ranges merge inside the launch, and the same without an exchange slot, on a distrusted exchange, on more streams
than there are slots and from a graph: the same bits everywhere, and the oracle's results.  Lists whose ranges don't merge inside a launch."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_17447_amd as fo
from paper_2605_17447_amd import binding as fb
from gpu_util import check_out, to_np
from test_gpu_sparse_layers import _launches, _layers, _one_by_one

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _merges(f):
    fb.kernel_timer_enable(fb.KERNEL_ATTN_COMBINE, 1024)
    try:
        f()
        torch.cuda.synchronize()
        return len(fb.kernel_timer_read(fb.KERNEL_ATTN_COMBINE))
    finally:
        fb.kernel_timer_enable(fb.KERNEL_ATTN_COMBINE, 0)


def _against_oracle(problem, outs, layers):
    batch, caches, qs, idx, cnt, _, scale = problem
    geo = [t.tolist() for t in (batch.seq_len, batch.vis_start, batch.vis_len)]
    for l in layers:
        c = caches[l]
        k, v = to_np(c.k), to_np(c.v)
        if c.block_table is None:
            cache = oracle.Cache.from_bhsd(k, v)
        else:
            pages, H, page, d = k.shape
            cache = oracle.Cache(k, v, H, d, stride_token=d, stride_head=page * d, page_tokens=page, stride_page=H * page * d,
                                 block_table=c.block_table.cpu().numpy())
        ref = oracle.decode_attn(cache, *geo, to_np(qs[l]), float(np.float32(scale)), idx.cpu().numpy(), cnt.cpu().numpy())
        check_out(outs[l], ref[0] if isinstance(ref, tuple) else ref, f"layer {l}")


@pytest.mark.parametrize("L,B,Hq,Hkv,d,n,text,page", [
    (2, 1, 28, 4, 128, 4000, 700, 0),
    (5, 2, 28, 4, 128, 4000, 500, 16),
    (3, 3, 16, 2, 64, 6000, 1200, 0),
    (4, 1, 64, 8, 64, 6000, 900, 16),
])
def test_the_same_bits_with_and_without_an_exchange_slot(L, B, Hq, Hkv, d, n, text, page):
    problem = _layers(L, B, Hq, Hkv, d, n, text, page, seed=L)
    batch, caches, qs, idx, cnt, ws, scale = problem

    def run(stream=None):
        outs = [torch.full_like(q, 5.0) for q in qs]
        torch.cuda.synchronize()
        fb.sparse_decode_attn_layers(caches, batch, qs, scale, idx, cnt, outs, ws, stream=stream)
        return outs

    want = []
    assert _launches(lambda: want.extend(run())) == 1 and _merges(run) == 0        # several ranges per stream: see the fallback's merges below
    _against_oracle(problem, want, {0, L - 1})
    got = []
    fb.set_tuning("exchange_fallback", 1)
    try:
        assert _merges(lambda: got.extend(run())) == L
    finally:
        fb.set_tuning("exchange_fallback", 0)
    assert all(torch.equal(a, b) for a, b in zip(got, want)), "distrusted exchange"
    streams = [torch.cuda.Stream() for _ in range(8)]
    for st in streams:
        fb.stream_release(st)
    try:
        def on_all():
            for i, st in enumerate(streams):
                res = run(st)
                st.synchronize()
                assert all(torch.equal(a, b) for a, b in zip(res, want)), f"stream {i}"
        assert 0 < _merges(on_all) < len(streams) * L                              # the first ones have slots, the last ones none
    finally:
        for st in streams:
            fb.stream_release(st)


@pytest.mark.parametrize("fallback", [0, 1])
@pytest.mark.parametrize("L,B,Hq,Hkv,d,n,text,page", [(3, 2, 28, 4, 128, 4000, 500, 16), (4, 1, 16, 2, 64, 6000, 1200, 0),
                                                      (6, 2, 28, 4, 128, 300, 60, 0), (5, 9, 64, 8, 128, 500, 200, 16), (5, 8, 64, 8, 64, 300, 200, 0)])
def test_a_captured_set_of_layers_replays_like_the_eager_one(L, B, Hq, Hkv, d, n, text, page, fallback):
    """Ranges that merge inside the launch, one range in eight waves, and more streams than compute units (four waves), from a graph that is
    replayed over changing queries and sets."""
    problem = _layers(L, B, Hq, Hkv, d, n, text, page, seed=7 + L)
    batch, caches, qs, idx, cnt, ws, scale = problem
    outs = [torch.zeros_like(q) for q in qs]
    call = lambda o: fb.sparse_decode_attn_layers(caches, batch, qs, scale, idx, cnt, o, ws)       # noqa: E731
    fb.set_tuning("exchange_fallback", fallback)
    try:
        call(outs)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            call(outs)
        gen = torch.Generator(device=DEV).manual_seed(1)
        for _ in range(4):
            for q in qs:
                q.copy_(torch.randn(q.shape, generator=gen, device=DEV))
            idx.copy_((idx + 1) % batch.vis_len[:, None])                          # distinct entries stay distinct
            eager = [torch.zeros_like(q) for q in qs]
            call(eager)
            torch.cuda.synchronize()
            for o in outs:
                o.fill_(9.0)
            graph.replay()
            torch.cuda.synchronize()
            assert all(torch.equal(a, b) for a, b in zip(outs, eager))
        _against_oracle(problem, outs, {0, L - 1})
    finally:
        fb.set_tuning("exchange_fallback", 0)


@pytest.mark.parametrize("L,rows,launches", [(2, 70, 2), (3, 70, 1), (3, 90, 3), (6, 140, 1)])
def test_long_lists_in_groups_of_more_heads_than_the_merge_takes(L, rows, launches):
    """16 query heads per kv head: one range per stream in one launch up to 24 tiles a layer, the layers' own calls beyond that."""
    text = 32 * rows - 50
    problem = _layers(L, 2, 16, 1, 128, 1000, text, ragged=False, seed=rows)
    batch, caches, qs, idx, cnt, ws, scale = problem
    assert text + idx.size(1) <= 32 * rows and text + idx.size(1) > 32 * (rows - 1)
    want = _one_by_one(batch, caches, qs, idx, cnt, ws, scale, [torch.zeros_like(q) for q in qs])
    outs = [torch.full_like(q, 5.0) for q in qs]
    assert _launches(lambda: fb.sparse_decode_attn_layers(caches, batch, qs, scale, idx, cnt, outs, ws)) == launches
    if launches == L:
        assert all(torch.equal(a, b) for a, b in zip(outs, want))
    _against_oracle(problem, outs, {0, L - 1})
