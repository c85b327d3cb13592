"""Layers whose output lies in the keys, values or pages that another layer attends: they run in their order, with the results of their own
calls."""
import pytest
import torch

import paper_2605_17447_amd as fo
from paper_2605_17447_amd import binding as fb
from test_gpu_sparse_layers import _launches, _layers, _one_by_one

pytestmark = pytest.mark.gpu


def _twin(caches):
    return [fo.KvCache(c.k.clone(), c.v.clone(), c.layout, c.block_table) for c in caches]


@pytest.mark.parametrize("page", [0, 16])
@pytest.mark.parametrize("writer,reader,which", [(0, 1, "k"), (0, 2, "v"), (1, 2, "k"), (2, 0, "v")])
@pytest.mark.parametrize("native", [True, False])
def test_an_output_in_another_layers_cache(page, writer, reader, which, native, monkeypatch):
    batch, caches, qs, idx, cnt, ws, scale = _layers(3, 2, 28, 4, 128, 300, 60, page, ragged=False, seed=9)
    if not native:
        monkeypatch.setattr(fb, "_call", None)
    results = []
    for together in (False, True):
        mine = _twin(caches)
        outs = [torch.zeros_like(q) for q in qs]
        pool = getattr(mine[reader], which).view(-1)
        first = int(mine[reader].block_table[0, 0]) * 4 * page * 128 if page else 0         # the first sequence's first rows: text before its image
        outs[writer] = pool[first: first + outs[0].numel()].view_as(outs[0])
        if together:
            assert _launches(lambda: fb.sparse_decode_attn_layers(mine, batch, qs, scale, idx, cnt, outs, ws)) == 3
        else:
            _one_by_one(batch, mine, qs, idx, cnt, ws, scale, outs)
        torch.cuda.synchronize()
        results.append([t.clone() for t in outs] + [getattr(c, x).clone() for c in mine for x in "kv"])
    assert all(torch.equal(a, b) for a, b in zip(*results))
    # (the writer's output changed what the reader attended, so that the order counts)
    plain = _one_by_one(batch, _twin(caches), qs, idx, cnt, ws, scale, [torch.zeros_like(q) for q in qs])
    assert torch.equal(plain[reader], results[0][reader]) == (writer > reader)
