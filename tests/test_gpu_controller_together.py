"""The step controller over runs of several pruned layers: with every query at hand (layers in shared launches), eager against a replayed graph,
bit for bit, and each output against the oracle; with queries that are made from the layer before, against the same calls in order."""
import numpy as np
import pytest
import torch

import fastocr_synth as fs
import oracle
import paper_2605_17447_amd as fo

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from gpu_util import DEV, check_out

L, FOCAL, TAU, STEPS = 9, (2, 6), 0.1, 6


@pytest.fixture(scope="module")
def stack():
    wl = fs.config(3, batch=2, n_layers=L, focal_layers=FOCAL, steps=STEPS, warmup=0, n_visual=(1024, 1024), grid_w=(32, 32), text_prefix=(30, 30))
    bts = [fs.make_batch(wl, device=DEV, layer=l) for l in range(L)]
    return wl, bts, fs.centres(bts[0])


def _controller(stack):
    wl, bts, _ = stack
    bt = bts[0]
    return fo.FixationController([fo.KvCache(x.k, x.v) for x in bts], wl.n_q_heads, float(np.float32(wl.head_dim ** -0.5)), FOCAL, TAU, 0,
                                 max(bt.seq_len(STEPS)), max(bt.n_vis), wl.batch, DEV, focal_gap=1)


def _batch(stack, seq_len):
    bt = stack[1][0]
    i32 = lambda a: torch.tensor(list(a), dtype=torch.int32, device=DEV)                    # noqa: E731
    return fo.SeqBatch(seq_len, i32(bt.vis_start), i32(bt.n_vis), max(bt.seq_len(STEPS)), max(bt.n_vis))


def test_a_captured_step_with_runs_of_several_pruned_layers(stack):
    wl, bts, cs = stack
    queries = lambda t: [fs.queries_for_step(bts[l], t, [c[t - 1] for c in cs]) for l in range(L)]       # noqa: E731
    eager, graphed = _controller(stack), _controller(stack)
    seq_len = torch.tensor(bts[0].seq_len(1), dtype=torch.int32, device=DEV)
    batch = _batch(stack, seq_len)
    qs = [q.clone() for q in queries(1)]
    outs, ref = [torch.zeros_like(q) for q in qs], [torch.zeros_like(q) for q in qs]

    def load(t):
        seq_len.copy_(torch.tensor(bts[0].seq_len(t), dtype=torch.int32))
        for dst, src in zip(qs, queries(t)):
            dst.copy_(src)

    for t in (1, 2):
        load(t)
        eager.step(t, batch, qs, ref)
        graphed.step(t, batch, tuple(qs), tuple(outs))
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(ref, outs))
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        graphed.step(3, batch, qs, outs)
    for t in range(3, STEPS + 1):
        load(t)
        before = eager.kept_idx.cpu().numpy().copy(), eager.kept_cnt.cpu().numpy().copy()
        picked = {}
        eager.step(t, batch, qs, ref, on_select=lambda l, sc, idx, cnt: picked.__setitem__(l, (idx.cpu().numpy().copy(), cnt.cpu().numpy().copy())))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(ref, outs)), f"step {t}"
        assert torch.equal(eager.kept_idx, graphed.kept_idx) and torch.equal(eager.kept_cnt, graphed.kept_cnt)
        if t == STEPS:
            for l in range(L):
                kept = before if l < FOCAL[0] else picked[max(f for f in FOCAL if f <= l)]
                cache = oracle.Cache.from_bhsd(fs.to_oracle_array(bts[l].k), fs.to_oracle_array(bts[l].v))
                want = oracle.decode_attn(cache, bts[0].seq_len(t), bts[0].vis_start, bts[0].n_vis, fs.to_oracle_array(qs[l]),
                                          float(np.float32(wl.head_dim ** -0.5)), *(() if l in FOCAL else kept), n_threads=oracle.max_threads())
                check_out(outs[l], want[0], f"layer {l}")


@pytest.mark.parametrize("base", [object, list, tuple])
def test_queries_made_from_the_layer_before(stack, base):
    wl, bts, cs = stack
    first = fs.queries_for_step(bts[0], 2, [c[1] for c in cs])
    outs = [torch.zeros_like(first) for _ in range(L)]
    make = lambda before: torch.nn.functional.normalize(before.float(), dim=-1).mul(6.0).to(first.dtype)          # noqa: E731

    class Made(base):
        def __getitem__(self, l):
            return first if l == 0 else make(outs[l - 1])

    batch = _batch(stack, torch.tensor(bts[0].seq_len(2), dtype=torch.int32, device=DEV))
    ctl = _controller(stack)
    ctl.step(1, batch, Made(), outs)                                   # leaves a set
    start = ctl.kept_idx.clone(), ctl.kept_cnt.clone()
    ctl.step(2, batch, Made(), outs)
    got = [o.clone() for o in outs]
    # the same calls, one layer after the other
    idx, cnt, q = *start, first
    scores, ws = torch.zeros_like(ctl.scores), ctl._workspace(ctl.caches[0], batch)
    for l, cache in enumerate(ctl.caches):
        out = torch.zeros_like(first)
        if l in FOCAL:
            fo.focal_attn_score_topk(cache, batch, q, ctl.scale, TAU, out, scores, idx, cnt, ws, prev_idx=idx, prev_cnt=cnt)
        else:
            fo.sparse_decode_attn(cache, batch, q, ctl.scale, idx, cnt, out, ws)
        torch.cuda.synchronize()
        assert torch.equal(out, got[l]), f"layer {l}"
        q = make(out)
