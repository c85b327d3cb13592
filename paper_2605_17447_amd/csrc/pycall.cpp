// The binding's hot path in native code: one call of a step entry point from Python, its tensors checked and its views
// filled here instead of in Python and ctypes, which took 3.4 us per call (a launch takes the runtime 2.5 - 3): a pruned layer of a few
// hundred rows is bound by that, not by its 6 us kernel.
//
// Every function returns the library's status, or None when something is not as the plain case has it -- an object of another
// class, a tensor of the wrong type, shape or layout, no CUDA context yet, an exception: the caller then takes the
// Python path, which does the same call or raises what it always raised.  Nothing is kept from one call to the next.
#include <algorithm>
#include <deque>
#include <vector>

#include <torch/csrc/autograd/python_variable.h>

#include "apart.hpp"
#include "fastocr.h"

namespace {

struct Library {
    decltype(&fastocr_focal_score) focal_score;
    decltype(&fastocr_topk_fixation) topk;
    decltype(&fastocr_sparse_decode_attn) sparse;
    decltype(&fastocr_dense_decode_attn) dense;
    decltype(&fastocr_focal_attn_score) layer;
    decltype(&fastocr_focal_score_topk) score_topk;
    decltype(&fastocr_focal_attn_score_topk) layer_topk;
} g_lib;
decltype(&fastocr_sparse_decode_attn_layers) g_sparse_layers = nullptr;
PyTypeObject *g_cache_type = nullptr, *g_batch_type = nullptr;
PyObject *g_device = nullptr, *g_raw_stream = nullptr, *g_initialized = nullptr;
PyObject *s_k, *s_v, *s_layout, *s_block_table, *s_seq_len, *s_vis_start, *s_vis_len, *s_max_seq_len, *s_max_vis_len, *s_cuda_stream;

// what sends a call back to the Python path
struct NotPlain {};
void require(bool ok) { if (!ok) throw NotPlain(); }

struct Ref {
    PyObject *p = nullptr;
    explicit Ref(PyObject *o) : p(o) { require(o != nullptr); }
    ~Ref() { Py_XDECREF(p); }
    Ref(const Ref &) = delete;
    Ref &operator=(const Ref &) = delete;
};

const at::Tensor &tensor(PyObject *o)
{
    require(THPVariable_CheckExact(o));
    return THPVariable_Unpack(o);
}
const at::Tensor &int32s(PyObject *o)
{
    const at::Tensor &t = tensor(o);
    require(t.scalar_type() == at::kInt);
    return t;
}
template <typename T = void>
T *optional(PyObject *o) { return o == Py_None ? nullptr : static_cast<T *>(tensor(o).data_ptr()); }
template <typename T = void>
T *data(const at::Tensor &t) { return static_cast<T *>(t.data_ptr()); }

double number(PyObject *o)
{
    require(PyFloat_CheckExact(o) || PyLong_CheckExact(o));
    const double x = PyFloat_AsDouble(o);
    require(!(x == -1.0 && PyErr_Occurred()));
    return x;
}
int32_t whole(PyObject *o)
{
    require(PyLong_CheckExact(o));
    const long x = PyLong_AsLong(o);
    require(!(x == -1 && PyErr_Occurred()) && x >= INT32_MIN && x <= INT32_MAX);
    return (int32_t)x;
}

// The cache and batch objects' tensors, held while the call runs, and their C views.
struct Cache {
    Ref k, v, layout, table;
    fastocr_kv_view view{};
    explicit Cache(PyObject *o)
        : k(own(o, s_k)), v(PyObject_GetAttr(o, s_v)), layout(PyObject_GetAttr(o, s_layout)), table(PyObject_GetAttr(o, s_block_table))
    {
        const at::Tensor &K = tensor(k.p), &V = tensor(v.p);
        require(K.dim() == 4 && K.sizes() == V.sizes() && K.strides() == V.strides() && K.scalar_type() == V.scalar_type() && K.stride(3) == 1);
        require(K.scalar_type() == at::kFloat || K.scalar_type() == at::kBFloat16);
        view.k = K.data_ptr();
        view.v = V.data_ptr();
        view.dtype = K.scalar_type() == at::kBFloat16 ? FASTOCR_BF16 : FASTOCR_F32;
        view.head_dim = (int32_t)K.size(3);
        if (table.p != Py_None) {
            const at::Tensor &bt = int32s(table.p);
            require(bt.dim() == 2 && bt.is_contiguous());
            view.n_kv_heads = (int32_t)K.size(1);
            view.stride_token = K.stride(2);
            view.stride_head = K.stride(1);
            view.page_tokens = (int32_t)K.size(2);
            view.stride_page = K.stride(0);
            view.block_table = data<int32_t>(bt);
            view.max_pages_per_seq = (int32_t)bt.size(1);
            return;
        }
        require(PyUnicode_Check(layout.p));
        const bool heads_first = PyUnicode_CompareWithASCIIString(layout.p, "bhsd") == 0;
        require(heads_first || PyUnicode_CompareWithASCIIString(layout.p, "bshd") == 0);
        const int h = heads_first ? 1 : 2;
        view.n_kv_heads = (int32_t)K.size(h);
        view.stride_token = K.stride(3 - h);
        view.stride_head = K.stride(h);
        view.stride_seq = K.stride(0);
    }
    static PyObject *own(PyObject *o, PyObject *name)
    {
        require(Py_TYPE(o) == g_cache_type);
        return PyObject_GetAttr(o, name);
    }
};

struct Batch {
    Ref seq_len, vis_start, vis_len;
    fastocr_batch_view view{};
    explicit Batch(PyObject *o) : seq_len(own(o, s_seq_len)), vis_start(PyObject_GetAttr(o, s_vis_start)), vis_len(PyObject_GetAttr(o, s_vis_len))
    {
        const at::Tensor &a = int32s(seq_len.p), &b = int32s(vis_start.p), &c = int32s(vis_len.p);
        require(a.dim() >= 1 && a.sizes() == b.sizes() && a.sizes() == c.sizes() && a.is_contiguous() && b.is_contiguous() && c.is_contiguous());
        const Ref ms(PyObject_GetAttr(o, s_max_seq_len)), mv(PyObject_GetAttr(o, s_max_vis_len));
        view.batch = (int32_t)a.size(0);
        view.seq_len = data<int32_t>(a);
        view.vis_start = data<int32_t>(b);
        view.vis_len = data<int32_t>(c);
        view.max_seq_len = whole(ms.p);
        view.max_vis_len = whole(mv.p);
    }
    static PyObject *own(PyObject *o, PyObject *name)
    {
        require(Py_TYPE(o) == g_batch_type);
        return PyObject_GetAttr(o, name);
    }
};

void *stream_of(PyObject *stream)
{
    if (stream != Py_None) {
        const Ref h(PyObject_GetAttr(stream, s_cuda_stream));
        void *p = PyLong_AsVoidPtr(h.p);
        require(!PyErr_Occurred());
        return p;
    }
    const Ref up(PyObject_CallNoArgs(g_initialized));
    require(up.p == Py_True);
    const Ref dev(PyObject_CallNoArgs(g_device));
    const Ref h(PyObject_CallOneArg(g_raw_stream, dev.p));
    void *p = PyLong_AsVoidPtr(h.p);
    require(!PyErr_Occurred());
    return p;
}

// q as the entry points take it; its query heads
int query_heads(const at::Tensor &q)
{
    require(q.dim() >= 2 && q.is_contiguous());
    return (int)q.size(1);
}
void *output(PyObject *o, const at::Tensor &q)
{
    const at::Tensor &t = tensor(o);
    require(t.is_contiguous() && t.sizes() == q.sizes() && t.scalar_type() == q.scalar_type());
    return t.data_ptr();
}
float *score_rows(PyObject *o, const fastocr_batch_view &bv, bool rows = true)
{
    const at::Tensor &t = tensor(o);
    require(t.dim() >= 2 && t.is_contiguous() && t.scalar_type() == at::kFloat);
    require((!rows || t.size(0) == bv.batch) && (t.size(1) == bv.max_vis_len || bv.batch == 0));
    return data<float>(t);
}
// the selected set and the set of the step before
struct Sets {
    int32_t *idx, *cnt;
    const int32_t *prev_idx, *prev_cnt;
    int64_t kmax;
    Sets(PyObject *sel_idx, PyObject *sel_cnt, PyObject *pidx = Py_None, PyObject *pcnt = Py_None)
    {
        const at::Tensor &i = int32s(sel_idx);
        require(i.dim() >= 2 && i.is_contiguous());
        idx = data<int32_t>(i);
        cnt = data<int32_t>(int32s(sel_cnt));
        kmax = i.size(1);
        prev_idx = nullptr;
        if (pidx != Py_None) {
            const at::Tensor &p = int32s(pidx);
            require(p.is_contiguous() && p.sizes() == i.sizes());
            prev_idx = data<int32_t>(p);
        }
        prev_cnt = optional<int32_t>(pcnt);
    }
};
struct Scratch {
    void *p;
    size_t bytes;
    explicit Scratch(PyObject *o) : p(nullptr), bytes(0)
    {
        if (o == Py_None) return;
        const at::Tensor &t = tensor(o);
        p = t.data_ptr();
        bytes = (size_t)t.numel();
    }
};

template <typename F>
PyObject *call(F f)
{
    try {
        return PyLong_FromLong(f());
    } catch (...) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}
// the library call itself, with the interpreter's lock released as ctypes does
template <typename F>
int unlocked(F f)
{
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f();
    Py_END_ALLOW_THREADS
    return rc;
}

#define FASTOCR_ARGS(N) if (n != (N)) { PyErr_SetString(PyExc_TypeError, "wrong number of arguments"); return nullptr; }

PyObject *focal_score(PyObject *, PyObject *const *a, Py_ssize_t n)          // cache, batch, q, scale, scores, ws, lse, img_mass, stream
{
    FASTOCR_ARGS(9)
    return call([&]() {
        require(a[5] != Py_None);
        const Cache c(a[0]);
        const Batch b(a[1]);
        const at::Tensor &q = tensor(a[2]);
        const int hq = query_heads(q);
        const float scale = (float)number(a[3]);
        float *scores = score_rows(a[4], b.view), *lse = optional<float>(a[6]), *mass = optional<float>(a[7]);
        const Scratch ws(a[5]);
        void *s = stream_of(a[8]), *qp = q.data_ptr();
        return unlocked([&]() { return g_lib.focal_score(&c.view, &b.view, qp, hq, scale, scores, lse, mass, ws.p, ws.bytes, s); });
    });
}

PyObject *topk(PyObject *, PyObject *const *a, Py_ssize_t n)                 // scores, batch, tau, sel_idx, sel_cnt, ws, prev_idx, prev_cnt, stream
{
    FASTOCR_ARGS(9)
    return call([&]() {
        const Batch b(a[1]);
        float *scores = score_rows(a[0], b.view, false);
        const double tau = number(a[2]);
        const Sets k(a[3], a[4], a[6], a[7]);
        const Scratch ws(a[5]);
        void *s = stream_of(a[8]);
        return unlocked([&]() { return g_lib.topk(scores, &b.view, tau, k.prev_idx, k.prev_cnt, k.idx, k.cnt, k.kmax, ws.p, ws.bytes, s); });
    });
}

PyObject *sparse(PyObject *, PyObject *const *a, Py_ssize_t n)               // cache, batch, q, scale, sel_idx, sel_cnt, out, ws, stream
{
    FASTOCR_ARGS(9)
    return call([&]() {
        require(a[7] != Py_None);
        const Cache c(a[0]);
        const Batch b(a[1]);
        const at::Tensor &q = tensor(a[2]);
        const int hq = query_heads(q);
        const float scale = (float)number(a[3]);
        const Sets k(a[4], a[5]);
        const Scratch ws(a[7]);
        void *out = output(a[6], q), *s = stream_of(a[8]), *qp = q.data_ptr();
        return unlocked([&]() { return g_lib.sparse(&c.view, &b.view, qp, hq, scale, k.idx, k.cnt, k.kmax, out, ws.p, ws.bytes, s); });
    });
}

// the bytes between which a tensor's elements lie
fastocr::Span reach(const at::Tensor &t)
{
    int64_t last = 1;
    for (int64_t i = 0; i < t.dim(); ++i) last += (t.size(i) - 1) * t.stride(i);
    return fastocr::span_of(t.data_ptr(), t.numel() ? last * (int64_t)t.element_size() : 0);
}

PyObject *sparse_layers(PyObject *, PyObject *const *a, Py_ssize_t n)        // caches, batch, queries, scale, sel_idx, sel_cnt, outs, ws, stream
{
    FASTOCR_ARGS(9)
    return call([&]() {
        require(g_sparse_layers != nullptr && a[7] != Py_None && PyList_CheckExact(a[0]) && PyList_CheckExact(a[2]) && PyList_CheckExact(a[6]));
        const Py_ssize_t m = PyList_GET_SIZE(a[0]);
        require(m > 0 && PyList_GET_SIZE(a[2]) == m && PyList_GET_SIZE(a[6]) == m);
        const Batch b(a[1]);
        const float scale = (float)number(a[3]);
        const Sets k(a[4], a[5]);
        const Scratch ws(a[7]);
        void *s = stream_of(a[8]);
        std::deque<Cache> caches;
        std::vector<fastocr_kv_view> views;
        std::vector<const void *> q;
        std::vector<void *> out;
        int hq = 0;
        for (Py_ssize_t l = 0; l < m; ++l) {
            views.push_back(caches.emplace_back(PyList_GET_ITEM(a[0], l)).view);
            const at::Tensor &t = tensor(PyList_GET_ITEM(a[2], l));
            require(l == 0 || query_heads(t) == hq);
            hq = query_heads(t);
            q.push_back(t.data_ptr());
            out.push_back(output(PyList_GET_ITEM(a[6], l), t));
        }
        // an output in the pool of a paged cache, whose reach the library does not know, is left to the Python path
        std::vector<fastocr::Span> pools;
        for (const Cache &c : caches) if (c.table.p != Py_None) for (PyObject *t : {c.k.p, c.v.p}) pools.push_back(reach(tensor(t)));
        if (!pools.empty()) {
            std::sort(pools.begin(), pools.end(), [](const fastocr::Span &x, const fastocr::Span &y) { return x.lo < y.lo; });
            // (pools that share memory: a span up to the farthest end so far)
            for (size_t i = 1; i < pools.size(); ++i) pools[i].hi = std::max(pools[i].hi, pools[i - 1].hi);
            for (Py_ssize_t l = 0; l < m; ++l) {
                const fastocr::Span o = reach(tensor(PyList_GET_ITEM(a[6], l)));
                const auto p = std::partition_point(pools.begin(), pools.end(), [&](const fastocr::Span &x) { return x.lo < o.hi; });
                require(p == pools.begin() || std::prev(p)->hi <= o.lo);
            }
        }
        return unlocked([&]() {
            return g_sparse_layers((int)m, views.data(), &b.view, q.data(), hq, scale, k.idx, k.cnt, k.kmax, out.data(), ws.p, ws.bytes, s);
        });
    });
}

// bind_layers(address of fastocr_sparse_decode_attn_layers)
PyObject *bind_layers(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    FASTOCR_ARGS(1)
    void *f = PyLong_AsVoidPtr(a[0]);
    if (PyErr_Occurred()) return nullptr;
    g_sparse_layers = (decltype(g_sparse_layers))f;
    Py_RETURN_NONE;
}

PyObject *dense(PyObject *, PyObject *const *a, Py_ssize_t n)                // cache, batch, q, scale, out, ws, lse, stream
{
    FASTOCR_ARGS(8)
    return call([&]() {
        require(a[5] != Py_None);
        const Cache c(a[0]);
        const Batch b(a[1]);
        const at::Tensor &q = tensor(a[2]);
        const int hq = query_heads(q);
        const float scale = (float)number(a[3]);
        const Scratch ws(a[5]);
        float *lse = optional<float>(a[6]);
        void *out = output(a[4], q), *s = stream_of(a[7]), *qp = q.data_ptr();
        return unlocked([&]() { return g_lib.dense(&c.view, &b.view, qp, hq, scale, out, lse, ws.p, ws.bytes, s); });
    });
}

PyObject *layer(PyObject *, PyObject *const *a, Py_ssize_t n)                // cache, batch, q, scale, out, scores, ws, lse, img_mass, stream
{
    FASTOCR_ARGS(10)
    return call([&]() {
        require(a[6] != Py_None);
        const Cache c(a[0]);
        const Batch b(a[1]);
        const at::Tensor &q = tensor(a[2]);
        const int hq = query_heads(q);
        const float scale = (float)number(a[3]);
        float *scores = score_rows(a[5], b.view), *lse = optional<float>(a[7]), *mass = optional<float>(a[8]);
        const Scratch ws(a[6]);
        void *out = output(a[4], q), *s = stream_of(a[9]), *qp = q.data_ptr();
        return unlocked([&]() { return g_lib.layer(&c.view, &b.view, qp, hq, scale, out, scores, lse, mass, ws.p, ws.bytes, s); });
    });
}

PyObject *score_topk(PyObject *, PyObject *const *a, Py_ssize_t n)           // cache, batch, q, scale, tau, scores, sel_idx, sel_cnt, ws, prev_idx, prev_cnt, lse, img_mass, stream
{
    FASTOCR_ARGS(14)
    return call([&]() {
        require(a[8] != Py_None);
        const Cache c(a[0]);
        const Batch b(a[1]);
        const at::Tensor &q = tensor(a[2]);
        const int hq = query_heads(q);
        const float scale = (float)number(a[3]);
        const double tau = number(a[4]);
        float *scores = score_rows(a[5], b.view), *lse = optional<float>(a[11]), *mass = optional<float>(a[12]);
        const Sets k(a[6], a[7], a[9], a[10]);
        const Scratch ws(a[8]);
        void *s = stream_of(a[13]), *qp = q.data_ptr();
        return unlocked([&]() {
            return g_lib.score_topk(&c.view, &b.view, qp, hq, scale, tau, k.prev_idx, k.prev_cnt, k.idx, k.cnt, k.kmax, scores, lse, mass, ws.p, ws.bytes, s);
        });
    });
}

PyObject *layer_topk(PyObject *, PyObject *const *a, Py_ssize_t n)           // cache, batch, q, scale, tau, out, scores, sel_idx, sel_cnt, ws, prev_idx, prev_cnt, lse, img_mass, stream
{
    FASTOCR_ARGS(15)
    return call([&]() {
        require(a[9] != Py_None);
        const Cache c(a[0]);
        const Batch b(a[1]);
        const at::Tensor &q = tensor(a[2]);
        const int hq = query_heads(q);
        const float scale = (float)number(a[3]);
        const double tau = number(a[4]);
        float *scores = score_rows(a[6], b.view), *lse = optional<float>(a[12]), *mass = optional<float>(a[13]);
        const Sets k(a[7], a[8], a[10], a[11]);
        const Scratch ws(a[9]);
        void *out = output(a[5], q), *s = stream_of(a[14]), *qp = q.data_ptr();
        return unlocked([&]() {
            return g_lib.layer_topk(&c.view, &b.view, qp, hq, scale, tau, k.prev_idx, k.prev_cnt, k.idx, k.cnt, k.kmax, out, scores, lse, mass, ws.p, ws.bytes, s);
        });
    });
}

// bind(cache type, batch type, current device, raw stream, is initialised, addresses of the seven entry points in Library's order)
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    FASTOCR_ARGS(12)
    if (!PyType_Check(a[0]) || !PyType_Check(a[1]) || !PyCallable_Check(a[2]) || !PyCallable_Check(a[3]) || !PyCallable_Check(a[4])) {
        PyErr_SetString(PyExc_TypeError, "bind: two types, three callables, seven addresses");
        return nullptr;
    }
    void *f[7];
    for (int i = 0; i < 7; ++i) {
        f[i] = PyLong_AsVoidPtr(a[5 + i]);
        if (PyErr_Occurred()) return nullptr;
    }
    for (int i = 0; i < 5; ++i) Py_INCREF(a[i]);             // kept for the life of the process
    g_cache_type = (PyTypeObject *)a[0];
    g_batch_type = (PyTypeObject *)a[1];
    g_device = a[2];
    g_raw_stream = a[3];
    g_initialized = a[4];
    g_lib = Library{(decltype(g_lib.focal_score))f[0], (decltype(g_lib.topk))f[1], (decltype(g_lib.sparse))f[2], (decltype(g_lib.dense))f[3],
                    (decltype(g_lib.layer))f[4], (decltype(g_lib.score_topk))f[5], (decltype(g_lib.layer_topk))f[6]};
    Py_RETURN_NONE;
}

#define FASTOCR_METHOD(NAME) {#NAME, (PyCFunction)(void (*)(void))NAME, METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {FASTOCR_METHOD(bind), FASTOCR_METHOD(focal_score), FASTOCR_METHOD(topk), FASTOCR_METHOD(sparse), FASTOCR_METHOD(dense),
                           FASTOCR_METHOD(layer), FASTOCR_METHOD(score_topk), FASTOCR_METHOD(layer_topk),
                           FASTOCR_METHOD(sparse_layers), FASTOCR_METHOD(bind_layers), {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_fastocr_call", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastocr_call()
{
    s_k = PyUnicode_InternFromString("k");
    s_v = PyUnicode_InternFromString("v");
    s_layout = PyUnicode_InternFromString("layout");
    s_block_table = PyUnicode_InternFromString("block_table");
    s_seq_len = PyUnicode_InternFromString("seq_len");
    s_vis_start = PyUnicode_InternFromString("vis_start");
    s_vis_len = PyUnicode_InternFromString("vis_len");
    s_max_seq_len = PyUnicode_InternFromString("max_seq_len");
    s_max_vis_len = PyUnicode_InternFromString("max_vis_len");
    s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    return PyModule_Create(&g_module);
}
