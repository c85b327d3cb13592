"""The native call path of the binding (csrc/pycall.cpp): the same arguments reach the library as through Python and ctypes, and
whatever is not the plain case is left to the Python path, which raises what it raises."""
import ctypes
import random
import types

import pytest
import torch

from paper_2605_17447_amd import binding as fb

fb.load_library()                                         # builds what is missing
_call = fb._call
if _call is None:
    if fb._raw_stream is None:
        pytest.skip("this torch has no stream handles to pass on", allow_module_level=True)
    raise RuntimeError("the library is built and its call extension is not")

P, I, I64, F, D, SZ = ctypes.c_void_p, ctypes.c_int, ctypes.c_int64, ctypes.c_float, ctypes.c_double, ctypes.c_size_t
KV, BV = ctypes.POINTER(fb.KvView), ctypes.POINTER(fb.BatchView)
SIGNATURES = {                                            # in the order bind() takes them
    "focal_score": [KV, BV, P, I, F, P, P, P, P, SZ, P],
    "topk_fixation": [P, BV, D, P, P, P, P, I64, P, SZ, P],
    "sparse_decode_attn": [KV, BV, P, I, F, P, P, I64, P, P, SZ, P],
    "dense_decode_attn": [KV, BV, P, I, F, P, P, P, SZ, P],
    "focal_attn_score": [KV, BV, P, I, F, P, P, P, P, P, SZ, P],
    "focal_score_topk": [KV, BV, P, I, F, D, P, P, P, P, I64, P, P, P, P, SZ, P],
    "focal_attn_score_topk": [KV, BV, P, I, F, D, P, P, P, P, I64, P, P, P, P, P, SZ, P],
}
STREAM = types.SimpleNamespace(cuda_stream=0x7000)


def _fields(x):
    if hasattr(x, "contents"):
        return tuple(getattr(x.contents, n) for n, *_ in x.contents._fields_)
    return x


@pytest.fixture
def both(monkeypatch):
    """run(name, *args, **kwargs) -> (what the native path passed on, what the Python path passed on); None: left to Python."""
    real = fb.load_library()
    seen, status = [], [0]

    def entry(name, sig):
        def f(*a):
            seen.append((name, tuple(_fields(x) for x in a)))
            return status[0]
        return ctypes.CFUNCTYPE(I, *sig)(f)

    entries = {n: entry(n, s) for n, s in SIGNATURES.items()}
    _call.bind(fb.KvCache, fb.SeqBatch, lambda: 3, lambda dev: 0x5000 + dev, lambda: True,
               *(ctypes.cast(e, P).value for e in entries.values()))
    lib = types.SimpleNamespace(**{"fastocr_" + n: e for n, e in entries.items()})
    none = types.SimpleNamespace()
    monkeypatch.setattr(fb, "load_library", lambda *a: real)
    monkeypatch.setattr(fb, "_lib", lib)
    monkeypatch.setattr(fb, "_stream_handle", lambda s: (0x5003 if s is None else s.cuda_stream) or None)

    def run(name, *args, rc=0, **kw):
        status[0] = rc
        out = []
        for native in (_call, None):
            monkeypatch.setattr(fb, "_call", native)
            monkeypatch.setattr(fb, "_lib", lib if native is None else none)          # (none: the Python path would not find its call)
            seen.clear()
            getattr(fb, name)(*args, **kw)
            out.append(list(seen))
        return out

    yield run, status, lib
    monkeypatch.undo()
    fb._bind_call(real)


def _problem(rng, dtype=torch.bfloat16):
    B, G, H, d = rng.randint(1, 4), rng.randint(1, 3), rng.randint(1, 3), rng.choice([64, 96, 128])
    S, N = rng.randint(40, 90), rng.randint(1, 40)
    layout = rng.choice(["bhsd", "bshd", "paged", "bhsd slices"])
    table = None
    if layout == "paged":
        k = torch.zeros(B * 6, H, 16, d, dtype=dtype)
        table = torch.zeros(B, 6, dtype=torch.int32)
    elif layout == "bshd":
        k = torch.zeros(B, S, H, d, dtype=dtype)
    elif layout == "bhsd":
        k = torch.zeros(B, H, S, d, dtype=dtype)
    else:                                                                # a view of a longer cache: odd strides
        k = torch.zeros(B + 1, H + 1, S + 7, d, dtype=dtype)[1:, :H, 3:3 + S]
        layout = "bhsd"
    v = k.clone() if k.is_contiguous() else torch.zeros(B + 1, H + 1, S + 7, d, dtype=dtype)[1:, :H, 3:3 + S]
    i32 = lambda *s: torch.zeros(*s, dtype=torch.int32)
    p = types.SimpleNamespace(cache=fb.KvCache(k, v, layout if table is None else "bhsd", table), batch=fb.SeqBatch(i32(B), i32(B), i32(B), S, N),
                              q=torch.zeros(B, H * G, d, dtype=dtype), out=torch.zeros(B, H * G, d, dtype=dtype), sc=torch.zeros(B, N),
                              idx=i32(B, 5), cnt=i32(B), pidx=i32(B, 5), pcnt=i32(B), lse=torch.zeros(B, H * G), mass=torch.zeros(B),
                              ws=torch.zeros(777, dtype=torch.uint8), scale=rng.choice([0.125, 1, 0.1]), tau=rng.choice([0.05, 0, 1]))
    return p


def _calls(p, opt):
    o = lambda t: t if opt else None
    st = STREAM if opt else None
    return [("focal_score", (p.cache, p.batch, p.q, p.scale, p.sc, p.ws), dict(lse=o(p.lse), img_mass=o(p.mass), stream=st)),
            ("topk_fixation", (p.sc, p.batch, p.tau, p.idx, p.cnt), dict(ws=o(p.ws), prev_idx=o(p.pidx), prev_cnt=o(p.pcnt), stream=st)),
            ("sparse_decode_attn", (p.cache, p.batch, p.q, p.scale, p.idx, p.cnt, p.out, p.ws), dict(stream=st)),
            ("dense_decode_attn", (p.cache, p.batch, p.q, p.scale, p.out, p.ws), dict(lse=o(p.lse), stream=st)),
            ("focal_attn_score", (p.cache, p.batch, p.q, p.scale, p.out, p.sc, p.ws), dict(lse=o(p.lse), img_mass=o(p.mass), stream=st)),
            ("focal_score_topk", (p.cache, p.batch, p.q, p.scale, p.tau, p.sc, p.idx, p.cnt, p.ws),
             dict(prev_idx=o(p.pidx), prev_cnt=o(p.pcnt), lse=o(p.lse), img_mass=o(p.mass), stream=st)),
            ("focal_attn_score_topk", (p.cache, p.batch, p.q, p.scale, p.tau, p.out, p.sc, p.idx, p.cnt, p.ws),
             dict(prev_idx=o(p.pidx), prev_cnt=o(p.pcnt), lse=o(p.lse), img_mass=o(p.mass), stream=st))]


@pytest.mark.parametrize("seed", range(12))
def test_the_same_arguments_reach_the_library(both, seed):
    run, _, _ = both
    rng = random.Random(seed)
    p = _problem(rng, torch.bfloat16 if seed % 2 else torch.float32)
    for opt in (False, True):
        for name, args, kw in _calls(p, opt):
            native, python = run(name, *args, **kw)
            assert len(native) == 1 and native == python, name


def test_a_status_is_raised_as_before(both):
    run, _, _ = both
    p = _problem(random.Random(1))
    for name, args, kw in _calls(p, False):
        with pytest.raises(fb.FastOcrError) as e:
            run(name, *args, rc=fb.EWORKSPACE, **kw)
        assert e.value.status == fb.EWORKSPACE and f"fastocr_{name}" in str(e.value)


def _broken():
    """(what, change): arguments the Python path refuses or treats in its own way."""
    t = lambda x: x.transpose(-1, -2) if x.dim() > 1 else x
    yield "query layout", lambda p: setattr(p, "q", t(torch.zeros(p.q.shape[0], p.q.shape[2], p.q.shape[1], dtype=p.q.dtype)))
    yield "output type", lambda p: setattr(p, "out", p.out.double())
    yield "output shape", lambda p: setattr(p, "out", p.out[:, :-1].contiguous())
    yield "set type", lambda p: setattr(p, "idx", p.idx.long())
    yield "set layout", lambda p: setattr(p, "idx", torch.zeros(5, p.idx.shape[0] + 1, dtype=torch.int32).t())
    yield "count type", lambda p: setattr(p, "cnt", p.cnt.long())
    yield "scores type", lambda p: setattr(p, "sc", p.sc.double())
    yield "scores pitch", lambda p: setattr(p, "sc", torch.zeros(p.sc.shape[0], p.sc.shape[1] + 1))
    yield "k and v differ", lambda p: setattr(p.cache, "v", p.cache.v[:, :, :-1])
    yield "cache type", lambda p: (setattr(p.cache, "k", p.cache.k.double()), setattr(p.cache, "v", p.cache.v.double()))
    yield "cache layout", lambda p: setattr(p.cache, "layout", "sbhd")
    yield "head dim strided", lambda p: (setattr(p.cache, "k", p.cache.k[..., ::2]), setattr(p.cache, "v", p.cache.v[..., ::2]))
    yield "lengths type", lambda p: setattr(p.batch, "seq_len", p.batch.seq_len.long())
    yield "lengths shape", lambda p: setattr(p.batch, "vis_len", torch.zeros(9, dtype=torch.int32))
    yield "a query that is no tensor", lambda p: setattr(p, "q", [1.0])
    yield "a scale that is no number", lambda p: setattr(p, "scale", "x")


@pytest.mark.parametrize("what,change", list(_broken()), ids=[w for w, _ in _broken()])
def test_what_is_not_plain_is_left_to_python(both, monkeypatch, what, change):
    _, _, lib = both
    p = next(p for p in (_problem(random.Random(s)) for s in range(99)) if min(p.q.shape[:2]) > 1 and p.sc.shape[1] > 1)
    if what == "cache layout":
        p.cache.block_table = None
    change(p)
    handled = 0
    for name, args, kw in _calls(p, True):
        results = []
        for call in (_call, None):
            monkeypatch.setattr(fb, "_call", call)
            try:
                getattr(fb, name)(*args, **kw)
                results.append(None)
            except Exception as e:                                       # noqa: BLE001
                results.append(type(e))
        assert results[0] == results[1], (name, results)
        handled += results[0] is not None
    assert handled > 0


def test_other_classes_and_subclasses_take_the_python_path(both, monkeypatch):
    run, _, lib = both
    p = _problem(random.Random(3))

    class Mine(fb.KvCache):
        pass

    class Sub(torch.Tensor):
        pass

    for cache, q in ((Mine(p.cache.k, p.cache.v, p.cache.layout, p.cache.block_table), p.q), (p.cache, p.q.as_subclass(Sub))):
        assert _call.sparse(cache, p.batch, q, p.scale, p.idx, p.cnt, p.out, p.ws, STREAM) is None
        monkeypatch.setattr(fb, "_call", _call)
        fb.sparse_decode_attn(cache, p.batch, q, p.scale, p.idx, p.cnt, p.out, p.ws, STREAM)
    assert _call.sparse(p.cache, p.batch, p.q, torch.tensor(0.5), p.idx, p.cnt, p.out, p.ws, STREAM) is None       # a scale Python converts
    with pytest.raises(TypeError):
        _call.sparse(p.cache)
