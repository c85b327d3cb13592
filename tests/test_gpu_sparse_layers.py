"""Pruned attention of several layers in one launch against the layers' own calls: one and several ranges per stream, more streams than
compute units, more layers than a launch takes, paged caches with a table per layer, and the lists that go through the calls one after
the other (unlike caches, fp32, an output where another layer's query or output lies)."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2605_17447_amd as fo
from paper_2605_17447_amd import binding as fb

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _layers(L, B, Hq, Hkv, d, n, text, page=0, dtype=torch.bfloat16, ragged=True, seed=0):
    g = torch.Generator(device=DEV).manual_seed(seed)
    rng = np.random.default_rng(seed)
    ns = [n if b == 0 or not ragged else int(rng.integers(1, n + 1)) for b in range(B)]
    ts = [text if not ragged else int(rng.integers(0, text + 1)) for _ in range(B)]
    seq = [a + t for a, t in zip(ns, ts)]
    S = max(seq)
    batch = fo.SeqBatch.from_lists(seq, [t // 2 for t in ts], ns, DEV)
    kmax = max(1, fo.keep_count(n, 0.05))
    idx = torch.full((B, kmax), 7, dtype=torch.int32)
    cnt = torch.zeros(B, dtype=torch.int32)
    for b, m in enumerate(ns):
        c = min(m, kmax if b % 3 else max(0, kmax - 3))
        idx[b, :c] = torch.from_numpy(np.sort(rng.permutation(m)[:c]).astype(np.int32))
        cnt[b] = c
    caches, qs = [], []
    for _ in range(L):
        if page:
            per = -(-S // page)
            table = torch.from_numpy(rng.permutation(B * per).astype(np.int32).reshape(B, per)).to(DEV)
            shape = (B * per, Hkv, page, d)
        else:
            table, shape = None, (B, Hkv, S, d)
        k, v = (torch.randn(shape, generator=g, device=DEV).to(dtype) for _ in range(2))
        caches.append(fo.KvCache(k, v, "bhsd", table))
        qs.append(torch.randn((B, Hq, d), generator=g, device=DEV).to(dtype))
    need = max(fo.workspace_bytes(fb.OP_SPARSE_DECODE_ATTN, c, batch, Hq, kmax) for c in caches)
    return batch, caches, qs, idx.to(DEV), cnt.to(DEV), torch.empty(max(need, 256), dtype=torch.uint8, device=DEV), d ** -0.5


def _one_by_one(batch, caches, qs, idx, cnt, ws, scale, outs):
    for c, q, o in zip(caches, qs, outs):
        fo.sparse_decode_attn(c, batch, q, scale, idx, cnt, o, ws)
    return outs


def _launches(f):
    fb.kernel_timer_enable(fb.KERNEL_SPARSE_ATTN, 256)
    try:
        f()
        torch.cuda.synchronize()
        return len(fb.kernel_timer_read(fb.KERNEL_SPARSE_ATTN))
    finally:
        fb.kernel_timer_enable(fb.KERNEL_SPARSE_ATTN, 0)


@pytest.mark.parametrize("L,B,Hq,Hkv,d,n,text,page,launches", [
    (2, 1, 28, 4, 128, 4000, 700, 0, 1),           # ranges merged inside the launch
    (7, 1, 16, 2, 64, 300, 40, 0, 1),              # one range, eight waves
    (5, 9, 64, 8, 128, 500, 200, 64, 1),           # more streams than compute units: four waves, a table per layer
    (3, 2, 12, 2, 64, 64, 3, 16, 1),
    (33, 3, 28, 4, 128, 200, 90, 0, 2),            # a layer more than a launch takes
    (2, 1, 16, 1, 128, 100, 20, 0, 1),             # sixteen heads per kv head
])
@pytest.mark.parametrize("native", [True, False])
def test_layers_in_one_launch(L, B, Hq, Hkv, d, n, text, page, launches, native, monkeypatch):
    batch, caches, qs, idx, cnt, ws, scale = _layers(L, B, Hq, Hkv, d, n, text, page, seed=L)
    want = _one_by_one(batch, caches, qs, idx, cnt, ws, scale, [torch.full_like(q, 3.0) for q in qs])
    if not native:
        monkeypatch.setattr(fb, "_call", None)
    outs = [torch.full_like(q, 5.0) for q in qs]
    assert _launches(lambda: fb.sparse_decode_attn_layers(caches, batch, qs, scale, idx, cnt, outs, ws)) == launches
    for l, (o, w) in enumerate(zip(outs, want)):
        o, w = o.float(), w.float()
        # two bf16 forms, each within 2e-2 of its row's maximum of the truth
        assert ((o - w).abs().amax(-1) <= 4e-2 * w.abs().amax(-1)).all(), l
        assert (o - w).norm() <= 1e-2 * w.norm(), l


def test_lists_that_go_through_the_calls_one_after_the_other():
    batch, caches, qs, idx, cnt, ws, scale = _layers(3, 2, 28, 4, 128, 700, 90, seed=5)
    want = _one_by_one(batch, caches, qs, idx, cnt, ws, scale, [torch.zeros_like(q) for q in qs])
    # an output in another layer's query: a later layer reads what an earlier one wrote
    chain = [qs[0].clone(), torch.zeros_like(qs[0]), torch.zeros_like(qs[0])]
    outs = [chain[1], chain[2], torch.zeros_like(qs[0])]
    ref = [qs[0].clone()]
    for c in caches:
        ref.append(torch.zeros_like(qs[0]))
        fo.sparse_decode_attn(c, batch, ref[-2], scale, idx, cnt, ref[-1], ws)
    assert _launches(lambda: fb.sparse_decode_attn_layers(caches, batch, chain, scale, idx, cnt, outs, ws)) == 3
    assert all(torch.equal(a, b) for a, b in zip(outs, ref[1:]))
    # one output for all: the last layer's stays
    same = torch.zeros_like(qs[0])
    fb.sparse_decode_attn_layers(caches, batch, qs, scale, idx, cnt, [same] * 3, ws)
    assert torch.equal(same, want[2])
    # caches of unlike strides, and fp32
    other = fo.KvCache(*(torch.cat([t, t], dim=2)[:, :, : t.size(2)] for t in (caches[1].k, caches[1].v)))
    outs = [torch.zeros_like(q) for q in qs]
    assert _launches(lambda: fb.sparse_decode_attn_layers([caches[0], other, caches[2]], batch, qs, scale, idx, cnt, outs, ws)) == 3
    assert all(torch.equal(a, b) for a, b in zip(outs, want))
    f32 = _layers(2, 2, 4, 2, 64, 90, 9, dtype=torch.float32)
    outs = [torch.zeros_like(q) for q in f32[2]]
    fb.sparse_decode_attn_layers(f32[1], f32[0], f32[2], f32[6], f32[3], f32[4], outs, f32[5])
    assert all(torch.equal(a, b) for a, b in zip(outs, _one_by_one(*f32, [torch.zeros_like(q) for q in f32[2]])))


def test_refused_before_anything_is_enqueued():
    batch, caches, qs, idx, cnt, ws, scale = _layers(2, 1, 4, 1, 128, 90, 9)
    outs = [torch.full_like(q, 5.0) for q in qs]
    lib, kv = fb.load_library(), (fb.KvView * 2)(caches[0].view(), caches[1].view())
    ptrs = lambda *a: (ctypes.c_void_p * 2)(*a)                                   # noqa: E731
    call = lambda n, kv, q, out, nb: lib.fastocr_sparse_decode_attn_layers(       # noqa: E731
        n, kv, ctypes.byref(batch.view()), q, 4, scale, idx.data_ptr(), cnt.data_ptr(), idx.size(1), out, ws.data_ptr(), nb, None)
    q, out = ptrs(*(x.data_ptr() for x in qs)), ptrs(*(x.data_ptr() for x in outs))
    kv[1].head_dim = 0
    assert call(2, kv, q, out, ws.numel()) == fb.EINVAL
    kv[1].head_dim = 128
    assert call(2, kv, ptrs(qs[0].data_ptr(), None), out, ws.numel()) == fb.EINVAL
    assert call(2, kv, q, ptrs(outs[0].data_ptr(), outs[1].data_ptr() + 2), ws.numel()) == fb.EINVAL
    assert call(2, kv, q, out, 0) == fb.EWORKSPACE
    assert call(-1, kv, q, out, ws.numel()) == fb.EINVAL and call(0, None, None, None, 0) == fb.OK
    torch.cuda.synchronize()
    assert all((o == 5.0).all() for o in outs)
