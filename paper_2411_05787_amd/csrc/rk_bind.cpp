// Argument marshalling of the short calls, in C++: what binding.py does for them one attribute at a time.
//
// Every function takes the binding's arguments in order, asks of every tensor what _dev() and _kv() ask
// (the plain class, device, type, contiguous or rows contiguous, shape) on every call, and returns the library's status; None if some
// argument is not as the common case has it, and nothing has been called then: binding.py goes through its own checks, for the message
// or the rarer form.  The interpreter lock is given up during the library's call, as ctypes does.
//
// A partial step of one layer over 256 rows takes the GPU 4.6 us; marshalled by Python and ctypes the host took 9.0.  An H2O step of 4 sequences of
// 2048 rows 22.2 -> 20.0.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>

#include <initializer_list>

#include "../../include/refreshkv.h"

namespace {

// binding.py's _stream, and the two functions of torch that give the current stream's handle (None where torch lacks them).
PyObject *g_stream, *g_raw_stream, *g_device;
// The ctypes classes of rk_geom and rk_h2o_state: what is of another class is binding.py's to refuse.
PyObject *g_geom, *g_h2o_state;

// One call's arguments: `ok` until one of them is not the common case's.
struct Args {
    PyObject* const* a;
    bool ok = true;
    rk_geom geom{};

    const at::Tensor* tensor(int i) {
        if (!ok || !THPVariable_CheckExact(a[i])) { ok = false; return nullptr; }
        const at::Tensor& t = THPVariable_Unpack(a[i]);
        if (!t.is_cuda()) { ok = false; return nullptr; }
        return &t;
    }
    void* dev(int i, at::ScalarType type, std::initializer_list<int64_t> shape) {
        const at::Tensor* t = tensor(i);
        if (!t) return nullptr;
        ok = t->scalar_type() == type && t->is_contiguous() && t->sizes() == at::IntArrayRef(shape);
        return ok ? t->data_ptr() : nullptr;
    }
    void* dev_or_null(int i, at::ScalarType type, std::initializer_list<int64_t> shape) {
        return a[i] == Py_None ? nullptr : dev(i, type, shape);
    }
    int64_t number(int i) {
        if (!ok || !PyLong_CheckExact(a[i])) { ok = false; return 0; }
        const long long v = PyLong_AsLongLong(a[i]);
        if (v == -1 && PyErr_Occurred()) { PyErr_Clear(); ok = false; }
        return v;
    }
    int32_t i32(int i) {
        const int64_t v = number(i);
        if (v < INT32_MIN || v > INT32_MAX) ok = false;
        return (int32_t)v;
    }
    // A ctypes structure by value.
    template <class T> T structure(PyObject* o, PyObject* type) {
        T s{};
        Py_buffer b;
        if (!ok || (PyObject*)Py_TYPE(o) != type || PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) { PyErr_Clear(); ok = false; return s; }
        ok = b.len == (Py_ssize_t)sizeof(T);
        if (ok) s = *(const T*)b.buf;
        PyBuffer_Release(&b);
        return s;
    }
    void geometry(int i) {                    // (Geom keeps its C structure once it has been asked for it)
        static PyObject* const name = PyUnicode_InternFromString("_c");
        PyObject* c = PyObject_GetAttr(a[i], name);
        if (!c) { PyErr_Clear(); ok = false; return; }
        geom = structure<rk_geom>(c, g_geom);
        Py_DECREF(c);
    }
    rk_kv kv(int k, int v, int64_t min_rows) {
        rk_kv r{};
        const at::Tensor *K = tensor(k), *V = tensor(v);
        if (!K || !V) return r;
        ok = K->scalar_type() == at::kBFloat16 && V->scalar_type() == at::kBFloat16 && K->dim() == 4 && V->sizes() == K->sizes() &&
             V->strides() == K->strides() && K->size(0) == geom.batch && K->size(1) == geom.n_kv_heads && K->size(3) == geom.head_dim &&
             K->stride(3) == 1 && K->stride(2) == geom.head_dim && K->size(2) >= min_rows;
        if (!ok) return r;
        return rk_kv{K->data_ptr(), V->data_ptr(), K->stride(0), K->stride(1), K->size(2)};
    }
    struct Scratch { void* ptr; size_t bytes; };
    Scratch workspace(int i) {
        static PyObject *const ptr = PyUnicode_InternFromString("ptr"), *const bytes = PyUnicode_InternFromString("nbytes");
        Scratch s{(void*)attribute(a[i], ptr), (size_t)attribute(a[i], bytes)};
        return s;
    }
    void* stream(int i) {                     // (asked for last, once every tensor is known to be in GPU memory)
        if (!ok || !g_stream) { ok = false; return nullptr; }
        PyObject *d = nullptr, *h = nullptr;
        if (a[i] != Py_None || g_raw_stream == Py_None || g_device == Py_None) {
            h = PyObject_CallFunctionObjArgs(g_stream, a[i], nullptr);
        } else if ((d = PyObject_CallNoArgs(g_device)) != nullptr) {
            h = PyObject_CallFunctionObjArgs(g_raw_stream, d, nullptr);
            Py_DECREF(d);
        }
        unsigned long long x = h && PyLong_Check(h) ? PyLong_AsUnsignedLongLong(h) : 0;
        if (!h || !PyLong_Check(h) || PyErr_Occurred()) { PyErr_Clear(); ok = false; }
        Py_XDECREF(h);
        return (void*)x;
    }

private:
    unsigned long long attribute(PyObject* o, PyObject* name) {
        PyObject* v = ok ? PyObject_GetAttr(o, name) : nullptr;
        unsigned long long x = 0;
        if (v && PyLong_CheckExact(v)) x = PyLong_AsUnsignedLongLong(v);
        if (!v || !PyLong_CheckExact(v) || PyErr_Occurred()) { PyErr_Clear(); ok = false; }
        Py_XDECREF(v);
        return x;
    }
};

template <class Call>
PyObject* status_of(Call&& call) {
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = call();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// Runs `body` on the arguments; None for a wrong number of them, or where a tensor has no memory to point at.
template <class Body>
PyObject* with_args(PyObject* const* a, Py_ssize_t n, Py_ssize_t want, Body&& body) {
    if (n != want) Py_RETURN_NONE;
    Args x{a};
    PyObject* r = nullptr;
    try {
        x.geometry(0);
        if (x.ok) r = body(x);
    } catch (...) {
        r = nullptr;
    }
    if (r) return r;
    PyErr_Clear();
    Py_RETURN_NONE;
}

constexpr auto bf16 = at::kBFloat16;
constexpr auto i32t = at::kInt;
constexpr auto f32 = at::kFloat;

// geom, q, small_K, small_V, n_sel, K, V, tail_start, seq_lens, max_recent, out, pred, pred_val, workspace, stream
template <int (*FN)(const rk_geom*, const void*, rk_kv, int32_t, rk_kv, const int32_t*, const int32_t*, int32_t, void*, const int32_t*, int32_t,
                    void*, size_t, void*)>
PyObject* partial(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return with_args(a, n, 15, [](Args& x) -> PyObject* {
        const rk_geom& g = x.geom;
        void* q = x.dev(1, bf16, {g.batch, g.n_q_heads, g.head_dim});
        const int32_t n_sel = x.i32(4), recent = x.i32(9), pred_val = x.i32(12);
        const rk_kv small = x.kv(2, 3, n_sel), full = x.kv(5, 6, 0);
        auto* tail = (const int32_t*)x.dev(7, i32t, {g.batch});
        auto* lens = (const int32_t*)x.dev(8, i32t, {g.batch});
        void* out = x.dev(10, bf16, {g.batch, g.n_q_heads, g.head_dim});
        auto* pred = (const int32_t*)x.dev_or_null(11, i32t, {g.batch});
        const Args::Scratch ws = x.workspace(13);
        void* st = x.stream(14);
        if (!x.ok) return nullptr;
        return status_of([&] { return FN(&g, q, small, n_sel, full, tail, lens, recent, out, pred, pred_val, ws.ptr, ws.bytes, st); });
    });
}

// geom, K, V, idx, k, small_K, small_V, seq_lens, tail_start, pred, pred_val, stream
PyObject* gather(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return with_args(a, n, 12, [](Args& x) -> PyObject* {
        const rk_geom& g = x.geom;
        const int32_t k = x.i32(4), pred_val = x.i32(10);
        const rk_kv full = x.kv(1, 2, 0), small = x.kv(5, 6, k);
        auto* idx = (const int32_t*)x.dev(3, i32t, {g.batch, g.n_kv_heads, k});
        auto* lens = (const int32_t*)x.dev_or_null(7, i32t, {g.batch});
        auto* tail = (int32_t*)x.dev_or_null(8, i32t, {g.batch});
        auto* pred = (const int32_t*)x.dev_or_null(9, i32t, {g.batch});
        void* st = x.stream(11);
        if (!x.ok) return nullptr;
        return status_of([&] { return rk_gather_small_kv(&g, full, idx, k, small, lens, tail, pred, pred_val, st); });
    });
}

// geom, state, q, k_new, v_new, seq_lens, budget, recent, out, agg, dropped, workspace, stream
PyObject* h2o_step(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return with_args(a, n, 13, [](Args& x) -> PyObject* {
        const rk_geom& g = x.geom;
        const rk_h2o_state state = x.structure<rk_h2o_state>(x.a[1], g_h2o_state);
        void* q = x.dev(2, bf16, {g.batch, g.n_q_heads, g.head_dim});
        void* k_new = x.dev(3, bf16, {g.batch, g.n_kv_heads, g.head_dim});
        void* v_new = x.dev(4, bf16, {g.batch, g.n_kv_heads, g.head_dim});
        auto* lens = (const int32_t*)x.dev(5, i32t, {g.batch});
        const int32_t budget = x.i32(6), recent = x.i32(7), agg = x.i32(9);
        void* out = x.dev(8, bf16, {g.batch, g.n_q_heads, g.head_dim});
        auto* dropped = (int32_t*)x.dev_or_null(10, i32t, {g.batch, g.n_kv_heads});
        const Args::Scratch ws = x.workspace(11);
        void* st = x.stream(12);
        if (!x.ok) return nullptr;
        return status_of([&] { return rk_h2o_step(&g, state, q, k_new, v_new, lens, budget, recent, agg, out, dropped, ws.ptr, ws.bytes, st); });
    });
}

// geom, q, K, V, seq_lens, max_len, out, lse, pred, pred_val, workspace, stream (no weights returned)
PyObject* full_attn(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return with_args(a, n, 12, [](Args& x) -> PyObject* {
        const rk_geom& g = x.geom;
        void* q = x.dev(1, bf16, {g.batch, g.n_q_heads, g.head_dim});
        const int32_t max_len = x.i32(5), pred_val = x.i32(9);
        const rk_kv full = x.kv(2, 3, max_len);
        auto* lens = (const int32_t*)x.dev(4, i32t, {g.batch});
        void* out = x.dev(6, bf16, {g.batch, g.n_q_heads, g.head_dim});
        auto* lse = (float*)x.dev_or_null(7, f32, {g.batch, g.n_q_heads});
        auto* pred = (const int32_t*)x.dev_or_null(8, i32t, {g.batch});
        const Args::Scratch ws = x.workspace(10);
        void* st = x.stream(11);
        if (!x.ok) return nullptr;
        return status_of([&] { return rk_full_attn(&g, q, full, lens, max_len, out, nullptr, 0, lse, pred, pred_val, ws.ptr, ws.bytes, st); });
    });
}

PyObject* setup(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 5) { PyErr_SetString(PyExc_TypeError, "setup(stream, raw_stream, device, geom, h2o_state)"); return nullptr; }
    for (int i = 0; i < 5; ++i) Py_INCREF(a[i]);
    g_stream = a[0]; g_raw_stream = a[1]; g_device = a[2]; g_geom = a[3]; g_h2o_state = a[4];
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"setup", (PyCFunction)(void (*)(void))setup, METH_FASTCALL, nullptr},
    {"rk_partial_attn", (PyCFunction)(void (*)(void))partial<rk_partial_attn>, METH_FASTCALL, nullptr},
    {"rk_partial_attn_fixed", (PyCFunction)(void (*)(void))partial<rk_partial_attn_fixed>, METH_FASTCALL, nullptr},
    {"rk_gather_small_kv", (PyCFunction)(void (*)(void))gather, METH_FASTCALL, nullptr},
    {"rk_h2o_step", (PyCFunction)(void (*)(void))h2o_step, METH_FASTCALL, nullptr},
    {"rk_full_attn", (PyCFunction)(void (*)(void))full_attn, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_rkbind", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__rkbind() { return PyModule_Create(&module); }
