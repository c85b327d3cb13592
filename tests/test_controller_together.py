"""When the step controller enqueues the pruned layers of a run together and when one by one (CPU only, on a recorder): plain lists hold
every layer's query, any other sequence may make one when it is asked for, from what the layers before it left."""
import pytest
import torch

from paper_2605_17447_amd.binding import SeqBatch
from paper_2605_17447_amd.controller import FixationController

_BATCH = SeqBatch.from_lists([300], [10], [256], "cpu")


class Recorder:
    """Records which layers' calls were enqueued, and what was asked of the queries in between."""

    def __init__(self):
        self.log = []

    def keep_count(self, n, tau):
        return max(1, int(n * tau))

    def workspace_bytes(self, *a, **k):
        return 256

    def dense_decode_attn(self, cache, batch, q, scale, out, ws, **kw):
        self.log.append(("dense", cache, q, out))

    def focal_attn_score_topk(self, cache, batch, q, scale, tau, out, *a, **kw):
        self.log.append(("focal", cache, q, out))

    def sparse_decode_attn(self, cache, batch, q, scale, sel_idx, sel_cnt, out, ws, **kw):
        self.log.append(("sparse", cache, q, out))

    def sparse_decode_attn_layers(self, caches, batch, queries, scale, sel_idx, sel_cnt, outs, ws, **kw):
        self.log.append(("layers", list(caches), list(queries), list(outs)))


class Asked:
    """A sequence of queries (of names, here) that writes down when one is asked for."""

    def _made(self, l):
        self.log.append(("asked", l))
        return f"q{l}"


class LazyList(Asked, list):
    def __getitem__(self, l):
        return self._made(l)


class LazyTuple(Asked, tuple):
    def __getitem__(self, l):
        return self._made(l)


class LazyOther(Asked):
    def __getitem__(self, l):
        return self._made(l)


def _controller(n_layers, focal):
    rec = Recorder()
    ctl = FixationController(list(range(n_layers)), 4, 0.125, focal, 0.05, 0, 300, 256, 1, "cpu", ops=rec)
    ctl.kept_from = "F_last"
    return rec, ctl


@pytest.mark.parametrize("kind", [LazyList, LazyTuple, LazyOther])
@pytest.mark.parametrize("which", ["queries", "outs"])
def test_a_layer_of_a_lazy_sequence_is_asked_for_once_and_after_the_call_before_it(kind, which):
    rec, ctl = _controller(6, [2])
    lazy, plain = kind(), [f"q{l}" for l in range(6)]
    lazy.log = rec.log
    ctl.step(1, _BATCH, *((lazy, plain) if which == "queries" else (plain, lazy)))
    calls = [("focal" if l == 2 else "sparse", l, f"q{l}", f"q{l}") for l in range(6)]
    assert rec.log == [x for l in range(6) for x in (("asked", l), calls[l])]


@pytest.mark.parametrize("kind", [list, tuple])
@pytest.mark.parametrize("n_layers,focal", [(6, [2]), (7, [0, 3]), (5, [4]), (4, [0, 2]), (1, [0])])
def test_plain_sequences_go_together_between_the_layers_that_select(kind, n_layers, focal):
    rec, ctl = _controller(n_layers, focal)
    qs, outs = kind(f"q{l}" for l in range(n_layers)), kind(f"o{l}" for l in range(n_layers))
    trace = ctl.step(1, _BATCH, qs, outs)
    want, run = [], []
    for l in range(n_layers + 1):
        if l < n_layers and l not in focal:
            run.append(l)
            continue
        if run:                                            # before the layer that writes the set anew
            want.append(("layers", run, [f"q{x}" for x in run], [f"o{x}" for x in run]))
            run = []
        if l < n_layers:
            want.append(("focal", l, f"q{l}", f"o{l}"))
    assert rec.log == want
    assert [m for _, m, _ in trace] == ["full+select" if l in focal else "pruned" for l in range(n_layers)]


def test_the_set_of_a_run_is_the_one_before_the_next_layer_selects():
    """on_select may write the queries of the layers that follow: those are read after it."""
    rec, ctl = _controller(5, [2])
    qs, outs = ["q0", "q1", "q2", None, None], [torch.zeros(1)] * 5

    def on_select(layer, scores, idx, cnt):
        assert [x[0] for x in rec.log] == ["layers", "focal"]
        qs[3], qs[4] = "q3", "q4"

    ctl.step(1, _BATCH, qs, outs, on_select=on_select)
    assert [(x[0], x[2]) for x in rec.log] == [("layers", ["q0", "q1"]), ("focal", "q2"), ("layers", ["q3", "q4"])]
