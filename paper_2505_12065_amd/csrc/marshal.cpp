// _marshal: what the binding's Python does for a call of the usual form (device tensors of the right types on the current device,
// outputs left to the binding), in native code.  Every function takes the binding's arguments with the current device and its stream
// behind them and returns what the entry point returns, the library's code if that is not 0, or None for a call of any other form,
// which the Python then takes, checks and answers or refuses.  Results are the same either way.
//
// A call on a small corpus is bound by the host: Python checks, two allocations and the conversions of a dozen arguments took 5.4 us of
// the 8.3 of a call of one launch (11.2 of two); here they take 1.9.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <torch/csrc/autograd/python_variable.h>

#include <initializer_list>

#include "../../include/ann.h"

namespace {

// the entry points of the library that the binding has loaded
decltype(&ann_flat_search_typed) flat_search;
decltype(&ann_flat_search_after_typed) flat_search_after;
decltype(&ann_graph_search_typed) graph_search;
decltype(&ann_graph_search_entries_typed) graph_search_entries;
decltype(&ann_graph_search_nonstall_typed) graph_search_nonstall;
decltype(&ann_gather_ids) gather_ids;
decltype(&ann_priority_order) priority_order;

struct OtherForm {};                                      // the call is not of the usual form

const at::Tensor &tensor(PyObject *o) {
    if (!THPVariable_CheckExact(o)) throw OtherForm();
    return THPVariable_Unpack(o);
}
// a contiguous device tensor with memory of its own
const at::Tensor &on_device(PyObject *o, int64_t device, at::ScalarType type) {
    const at::Tensor &t = tensor(o);
    if (!t.is_cuda() || t.get_device() != device || t.scalar_type() != type || !t.has_storage() ||
        t.unsafeGetTensorImpl()->is_python_dispatch() || !t.is_contiguous())
        throw OtherForm();
    return t;
}
int64_t integer(PyObject *o, int64_t least, int64_t most) {
    if (!PyLong_CheckExact(o)) throw OtherForm();
    int overflow = 0;
    const int64_t v = PyLong_AsLongLongAndOverflow(o, &overflow);
    if (overflow != 0 || v < least || v > most) throw OtherForm();
    return v;
}
int32_t int32(PyObject *o) { return (int32_t)integer(o, INT32_MIN, INT32_MAX); }
int32_t count(int64_t n) {
    if (n > INT32_MAX) throw OtherForm();
    return (int32_t)n;
}
void *stream_of(PyObject *o) {
    void *p = PyLong_AsVoidPtr(o);
    if (PyErr_Occurred()) {
        PyErr_Clear();
        throw OtherForm();
    }
    return p;
}

struct Call {                                             // corpus, queries and what they say
    int64_t device, N;
    int32_t d, dtype, B;
    const at::Tensor *x, *q;
    Call(PyObject *corpus, PyObject *queries, int64_t device_) : device(device_) {
        const at::ScalarType type = tensor(corpus).scalar_type();
        dtype = type == at::kHalf ? ANN_F16 : type == at::kBFloat16 ? ANN_BF16 : type == at::kFloat ? ANN_F32 : -1;
        if (dtype < 0) throw OtherForm();
        x = &on_device(corpus, device, type);
        q = &on_device(queries, device, type);
        if (x->dim() != 2 || q->dim() != 2 || x->size(1) != q->size(1)) throw OtherForm();
        N = x->size(0);
        d = count(x->size(1));
        B = count(q->size(0));
    }
};
at::Tensor empty(at::IntArrayRef size, at::ScalarType type, const at::Tensor &like) {
    return at::empty(size, at::TensorOptions().dtype(type).device(like.device()));
}
const int32_t *graph_of(PyObject *o, const Call &c, int32_t *R) {
    const at::Tensor &g = on_device(o, c.device, at::kInt);
    if (g.dim() != 2 || g.size(0) != c.N) throw OtherForm();
    *R = count(g.size(1));
    return static_cast<const int32_t *>(g.data_ptr());
}
const int32_t *entries_of(PyObject *o, const Call &c, int32_t *E) {
    const at::Tensor &e = on_device(o, c.device, at::kInt);
    if (!((e.dim() == 1 || (e.dim() == 2 && e.size(1) >= 1)) && e.size(0) == c.B)) throw OtherForm();
    *E = e.dim() == 1 ? 1 : count(e.size(1));
    return static_cast<const int32_t *>(e.data_ptr());
}
int32_t *ints(const at::Tensor &t) { return static_cast<int32_t *>(t.data_ptr()); }
float *floats(const at::Tensor &t) { return static_cast<float *>(t.data_ptr()); }

PyObject *answer(int code, std::initializer_list<const at::Tensor *> out) {
    if (code != ANN_OK) return PyLong_FromLong(code);
    PyObject *tuple = PyTuple_New((Py_ssize_t)out.size());
    if (!tuple) return nullptr;
    Py_ssize_t i = 0;
    for (const at::Tensor *t : out) {
        PyObject *o = THPVariable_Wrap(*t);
        if (!o) {
            Py_DECREF(tuple);
            return nullptr;
        }
        PyTuple_SET_ITEM(tuple, i++, o);
    }
    return tuple;
}

// body(args), and None where that says so, or meets an error: the Python gives it its name.
template <int N, class Body>
PyObject *usual(PyObject *const *args, Py_ssize_t n, Body &&body) {
    if (n != N || at::impl::torch_function_mode_enabled() || c10::impl::TorchDispatchModeTLS::any_modes_set()) Py_RETURN_NONE;
    try {
        return body(args);
    } catch (...) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}
template <class F, class... A>
int without_gil(F *f, A... a) {
    int code;
    Py_BEGIN_ALLOW_THREADS
    code = f(a...);
    Py_END_ALLOW_THREADS
    return code;
}

// corpus, queries, k, after scores, after ids (None, None: no boundary), device, stream
PyObject *flat(PyObject *, PyObject *const *args, Py_ssize_t n) {
    return usual<7>(args, n, [](PyObject *const *a) {
        const Call c(a[0], a[1], integer(a[5], 0, INT32_MAX));
        const int32_t k = int32(a[2]);
        const at::Tensor *s = nullptr, *i = nullptr;
        if (a[3] != Py_None || a[4] != Py_None) {
            s = &on_device(a[3], c.device, at::kFloat);
            i = &on_device(a[4], c.device, at::kInt);
            if (s->dim() != 1 || i->dim() != 1 || s->size(0) != c.B || i->size(0) != c.B) throw OtherForm();
        }
        void *stream = stream_of(a[6]);
        const at::Tensor ids = empty({c.B, k}, at::kInt, *c.x), scores = empty({c.B, k}, at::kFloat, *c.x);
        const int code = s ? without_gil(flat_search_after, c.x->data_ptr(), c.N, c.d, c.dtype, c.q->data_ptr(), c.B, k, floats(*s),
                                         ints(*i), ints(ids), floats(scores), stream)
                           : without_gil(flat_search, c.x->data_ptr(), c.N, c.d, c.dtype, c.q->data_ptr(), c.B, k, ints(ids),
                                         floats(scores), stream);
        return answer(code, {&ids, &scores});
    });
}

// corpus, graph, entry (ENTRIES: the tensor of one entry per query, else a number), queries, k, ef, device, stream
template <bool ENTRIES>
PyObject *graph_of_either(PyObject *, PyObject *const *args, Py_ssize_t n) {
    return usual<8>(args, n, [](PyObject *const *a) {
        const Call c(a[0], a[3], integer(a[6], 0, INT32_MAX));
        const int32_t k = int32(a[4]), ef = int32(a[5]);
        int32_t R, E = 0;
        const int32_t *g = graph_of(a[1], c, &R), *entries = nullptr;
        int32_t entry = 0;
        if (ENTRIES) {
            entries = entries_of(a[2], c, &E);
            if (tensor(a[2]).dim() != 1) throw OtherForm();
        } else {
            entry = int32(a[2]);
        }
        void *stream = stream_of(a[7]);
        const at::Tensor ids = empty({c.B, k}, at::kInt, *c.x), scores = empty({c.B, k}, at::kFloat, *c.x);
        const int code = ENTRIES ? without_gil(graph_search_entries, c.x->data_ptr(), c.N, c.d, c.dtype, g, R, entries, c.q->data_ptr(), c.B, k,
                                         ef, ints(ids), floats(scores), stream)
                                 : without_gil(graph_search, c.x->data_ptr(), c.N, c.d, c.dtype, g, R, entry, c.q->data_ptr(), c.B, k, ef,
                                         ints(ids), floats(scores), stream);
        return answer(code, {&ids, &scores});
    });
}

PyObject *graph(PyObject *self, PyObject *const *args, Py_ssize_t n) { return graph_of_either<false>(self, args, n); }
PyObject *graph_entries(PyObject *self, PyObject *const *args, Py_ssize_t n) { return graph_of_either<true>(self, args, n); }

// corpus, graph, entry, queries, k, ef, entries or None, tau, window, device, stream
PyObject *nonstall(PyObject *, PyObject *const *args, Py_ssize_t n) {
    return usual<11>(args, n, [](PyObject *const *a) {
        const Call c(a[0], a[3], integer(a[9], 0, INT32_MAX));
        const int32_t entry = int32(a[2]), k = int32(a[4]), ef = int32(a[5]), window = int32(a[8]);
        int32_t R, E = 0;
        const int32_t *g = graph_of(a[1], c, &R), *entries = a[6] != Py_None ? entries_of(a[6], c, &E) : nullptr;
        if (!PyFloat_CheckExact(a[7])) throw OtherForm();
        const float tau = (float)PyFloat_AS_DOUBLE(a[7]);
        void *stream = stream_of(a[10]);
        const at::Tensor ids = empty({c.B, k}, at::kInt, *c.x), scores = empty({c.B, k}, at::kFloat, *c.x),
                         stats = empty({c.B, 3}, at::kInt, *c.x), ema = empty({c.B}, at::kFloat, *c.x);
        const int code = without_gil(graph_search_nonstall, c.x->data_ptr(), c.N, c.d, c.dtype, g, R, entry, c.q->data_ptr(), c.B, k, ef,
                                     entries, E, tau, window, nullptr, ints(ids), floats(scores), ints(stats), floats(ema), stream);
        return answer(code, {&ids, &scores, &stats, &ema});
    });
}

// table, idx, device, stream
PyObject *gather(PyObject *, PyObject *const *args, Py_ssize_t n) {
    return usual<4>(args, n, [](PyObject *const *a) {
        const int64_t device = integer(a[2], 0, INT32_MAX);
        const at::Tensor &table = on_device(a[0], device, at::kInt), &idx = on_device(a[1], device, at::kInt);
        if (idx.dim() != 1) throw OtherForm();
        void *stream = stream_of(a[3]);
        const at::Tensor out = empty({idx.size(0)}, at::kInt, idx);
        return answer(without_gil(gather_ids, ints(table), table.numel(), ints(idx), idx.numel(), ints(out), stream), {&out});
    });
}

// R, W, C, Wcur, G, device, stream
PyObject *order(PyObject *, PyObject *const *args, Py_ssize_t n) {
    return usual<7>(args, n, [](PyObject *const *a) {
        const int64_t device = integer(a[5], 0, INT32_MAX);
        const at::Tensor &R = on_device(a[0], device, at::kInt), &W = on_device(a[1], device, at::kDouble),
                         &C = on_device(a[2], device, at::kInt), &Wcur = on_device(a[3], device, at::kDouble);
        const int32_t m = count(R.numel()), G = int32(a[4]);
        if (W.numel() != m || C.numel() != m || Wcur.numel() != m) throw OtherForm();
        void *stream = stream_of(a[6]);
        const at::Tensor level = empty({m}, at::kInt, R), rank = empty({m}, at::kInt, R);
        const int code = without_gil(priority_order, ints(R), static_cast<const double *>(W.data_ptr()), ints(C),
                                     static_cast<const double *>(Wcur.data_ptr()), m, G, ints(level), ints(rank), stream);
        return answer(code, {&level, &rank});
    });
}

// addresses of the entry points, in the order of their declarations above
PyObject *bind(PyObject *, PyObject *const *args, Py_ssize_t n) {
    void *p[7];
    if (n != 7) {
        PyErr_SetString(PyExc_TypeError, "bind takes 7 addresses");
        return nullptr;
    }
    for (int i = 0; i < 7; ++i) {
        p[i] = PyLong_AsVoidPtr(args[i]);
        if (PyErr_Occurred()) return nullptr;
    }
    flat_search = reinterpret_cast<decltype(flat_search)>(p[0]);
    flat_search_after = reinterpret_cast<decltype(flat_search_after)>(p[1]);
    graph_search = reinterpret_cast<decltype(graph_search)>(p[2]);
    graph_search_entries = reinterpret_cast<decltype(graph_search_entries)>(p[3]);
    graph_search_nonstall = reinterpret_cast<decltype(graph_search_nonstall)>(p[4]);
    gather_ids = reinterpret_cast<decltype(gather_ids)>(p[5]);
    priority_order = reinterpret_cast<decltype(priority_order)>(p[6]);
    Py_RETURN_NONE;
}

#define ENTRY(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {ENTRY(bind), ENTRY(flat), ENTRY(graph), ENTRY(graph_entries), ENTRY(nonstall), ENTRY(gather), ENTRY(order), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// (asks nothing of torch's objects: the binding looks at built_for before it binds)
PyMODINIT_FUNC PyInit__marshal() {
    PyObject *m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "built_for", ANN_BUILT_FOR) != 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
