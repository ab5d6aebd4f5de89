// The layer, flatten and retile calls as a Python extension module: arguments go from Python objects straight into the call's
// C arguments.  A training step of a small chain is six calls with 27 shard lists between them; through ctypes they took
// 44 us of host time, as long as the GPU needs for half the kernels, and so 12 us.
//
// Every function takes the address of the library's function first (the library itself knows nothing of Python).  What is
// accepted is what the ctypes binding accepts: shard lists are None (a NULL list) or sequences of objects with a data_ptr()
// or of integers; tilings and forms are strings, or whatever binding.tiling() / binding.forms() take.  The interpreter's
// lock is released during a call.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <cstring>
#include "tensor_tiling.h"

namespace {

constexpr int kMaxShards = 1 << TT_MAX_K;

PyObject *g_data_ptr, *g_numel, *g_element_size, *g_value; // method and attribute names
PyObject *g_tiling, *g_forms, *g_dtype;                     // the binding's own converters, for the rarer forms

// Arguments of one call.  The first failure leaves a Python exception set and every later step a no-op.
struct Args {
    PyObject *const *a;
    Py_ssize_t n, i = 0;
    bool ok = true;
    PyObject *held[8]; // objects whose buffers the call reads
    Py_buffer view[8];
    int n_held = 0, n_view = 0;

    Args(PyObject *const *args, Py_ssize_t nargs, Py_ssize_t want) : a(args), n(nargs)
    {
        if (n != want) {
            PyErr_Format(PyExc_TypeError, "%zd arguments expected, not %zd", want, n);
            ok = false;
        }
    }
    ~Args()
    {
        for (int v = 0; v < n_view; ++v) PyBuffer_Release(&view[v]);
        for (int h = 0; h < n_held; ++h) Py_DECREF(held[h]);
    }
    PyObject *next() { return ok ? a[i++] : nullptr; }
    bool fail() { return ok = false; }

    // an integer, wrapped to 64 bits as ctypes does
    uint64_t integer_of(PyObject *o)
    {
        PyObject *x = PyNumber_Index(o);
        if (!x) { fail(); return 0; }
        const uint64_t v = PyLong_AsUnsignedLongLongMask(x);
        Py_DECREF(x);
        if (v == ~0ull && PyErr_Occurred()) fail();
        return v;
    }
    int64_t i64() { PyObject *o = next(); return o ? (int64_t)integer_of(o) : 0; }
    int i32() { return (int)i64(); }
    template <class F> F address() { return reinterpret_cast<F>((uintptr_t)i64()); }
    int flag()
    {
        PyObject *o = next();
        if (!o) return 0;
        const int v = PyObject_IsTrue(o);
        if (v < 0) fail();
        return v > 0;
    }
    // bytes of a ctypes object, valid until the call is over
    const void *bytes_of(PyObject *o, Py_ssize_t least)
    {
        if (n_view == 8 || PyObject_GetBuffer(o, &view[n_view], PyBUF_SIMPLE) != 0) { fail(); return nullptr; }
        const Py_buffer &v = view[n_view++];
        if (v.len < least) {
            PyErr_SetString(PyExc_TypeError, "structure of another type");
            fail();
            return nullptr;
        }
        return v.buf;
    }
    PyObject *converted(PyObject *converter, PyObject *o) // kept until the call is over
    {
        PyObject *x = n_held < 8 ? PyObject_CallOneArg(converter, o) : nullptr;
        if (!x) { fail(); return nullptr; }
        return held[n_held++] = x;
    }
    const tt_layer *layer()
    {
        PyObject *o = next();
        return o ? static_cast<const tt_layer *>(bytes_of(o, sizeof(tt_layer))) : nullptr;
    }
    tt_tiling tiling()
    {
        tt_tiling t;
        std::memset(&t, 0, sizeof(t));
        PyObject *o = next();
        if (!o) return t;
        if (PyUnicode_CheckExact(o) && PyUnicode_GET_LENGTH(o) <= TT_MAX_K) {
            for (Py_ssize_t j = 0; j < PyUnicode_GET_LENGTH(o); ++j) {
                const Py_UCS4 c = PyUnicode_READ_CHAR(o, j);
                t.cut[j] = c == 'R' ? TT_R : c == 'C' ? TT_C : c == 'r' ? TT_REP : 255;
            }
            return t;
        }
        PyObject *x = converted(g_tiling, o);
        if (const void *b = x ? bytes_of(x, sizeof(t)) : nullptr) std::memcpy(&t, b, sizeof(t));
        return t;
    }
    const uint8_t *forms(uint8_t (&buf)[TT_MAX_K])
    {
        PyObject *o = next();
        if (!o || o == Py_None) return nullptr;
        std::memset(buf, 255, sizeof(buf)); // (no form: a sequence shorter than k is refused)
        if (PyUnicode_CheckExact(o) && PyUnicode_GET_LENGTH(o) <= TT_MAX_K) {
            Py_ssize_t j = 0;
            for (; j < PyUnicode_GET_LENGTH(o); ++j) {
                const Py_UCS4 c = PyUnicode_READ_CHAR(o, j);
                if (c < '1' || c > '9') break;
                buf[j] = (uint8_t)(c - '1');
            }
            if (j == PyUnicode_GET_LENGTH(o)) return buf;
        }
        PyObject *x = converted(g_forms, o);
        return x ? static_cast<const uint8_t *>(bytes_of(x, TT_MAX_K)) : nullptr; // (the converter fills up short sequences)
    }
    int dtype()
    {
        PyObject *o = next();
        if (!o) return 0;
        if (PyUnicode_CheckExact(o)) {
            if (PyUnicode_CompareWithASCIIString(o, "bf16") == 0) return TT_BF16;
            if (PyUnicode_CompareWithASCIIString(o, "f32") == 0) return TT_F32;
        }
        PyObject *x = converted(g_dtype, o);
        return x ? (int)integer_of(x) : 0;
    }
    uint64_t pointer_of(PyObject *o)
    {
        PyObject *p = PyObject_CallMethodNoArgs(o, g_data_ptr);
        if (!p) {
            if (!PyErr_ExceptionMatches(PyExc_AttributeError)) { fail(); return 0; }
            PyErr_Clear();
            p = PyNumber_Long(o);
            if (!p) { fail(); return 0; }
        }
        const uint64_t v = integer_of(p);
        Py_DECREF(p);
        return v;
    }
    // a shard list; entries past the last one given are NULL
    void **shards(void *(&buf)[kMaxShards])
    {
        PyObject *o = next();
        if (!o || o == Py_None) return nullptr;
        PyObject *s = PySequence_Fast(o, "a shard list is a sequence");
        if (!s) { fail(); return nullptr; }
        for (Py_ssize_t j = 0; j < kMaxShards; ++j) { // (data_ptr() is Python code: the length is read anew)
            buf[j] = nullptr;
            if (!ok || j >= PySequence_Fast_GET_SIZE(s)) continue;
            PyObject *item = PySequence_Fast_GET_ITEM(s, j);
            Py_INCREF(item);
            buf[j] = reinterpret_cast<void *>((uintptr_t)pointer_of(item));
            Py_DECREF(item);
        }
        Py_DECREF(s);
        return buf;
    }
    uint64_t method(PyObject *o, PyObject *name)
    {
        PyObject *x = PyObject_CallMethodNoArgs(o, name);
        if (!x) { fail(); return 0; }
        const uint64_t v = integer_of(x);
        Py_DECREF(x);
        return v;
    }
    void *workspace(size_t *bytes)
    {
        *bytes = 0;
        PyObject *o = next();
        if (!o || o == Py_None) return nullptr;
        const uint64_t p = method(o, g_data_ptr);
        if (ok) *bytes = (size_t)method(o, g_numel);
        if (ok) *bytes *= (size_t)method(o, g_element_size);
        return reinterpret_cast<void *>((uintptr_t)p);
    }
    // a handle: an integer, None or a ctypes pointer
    void *stream()
    {
        PyObject *o = next();
        if (!o || o == Py_None) return nullptr;
        if (PyLong_CheckExact(o)) return reinterpret_cast<void *>((uintptr_t)integer_of(o));
        PyObject *v = PyObject_GetAttr(o, g_value);
        if (!v) { fail(); return nullptr; }
        void *p = v == Py_None ? nullptr : reinterpret_cast<void *>((uintptr_t)integer_of(v));
        Py_DECREF(v);
        return p;
    }
};

template <class F> PyObject *finish(Args &g, F &&call)
{
    if (!g.ok) return nullptr;
    tt_status st;
    Py_BEGIN_ALLOW_THREADS
    st = call();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong((long)st);
}

const void *const *in(void **p) { return const_cast<const void *const *>(p); }

// forward(address, layer, batch, k, dtype, tX, tW, tY, forms, X, W, Y, workspace, stream): tt_fc_forward, tt_conv_forward
PyObject *forward(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    Args g(args, n, 14);
    auto fn = g.address<decltype(&tt_fc_forward)>();
    const tt_layer *lay = g.layer();
    const int64_t batch = g.i64();
    const int k = g.i32(), dt = g.dtype();
    const tt_tiling tX = g.tiling(), tW = g.tiling(), tY = g.tiling();
    uint8_t fb[TT_MAX_K];
    void *x[kMaxShards], *w[kMaxShards], *y[kMaxShards];
    const uint8_t *f = g.forms(fb);
    void **X = g.shards(x), **W = g.shards(w), **Y = g.shards(y);
    size_t bytes;
    void *ws = g.workspace(&bytes), *stream = g.stream();
    return finish(g, [&] { return fn(lay, batch, k, dt, tX, tW, tY, f, in(X), in(W), Y, ws, bytes, stream); });
}

// forward_static(address, layer, batch, k, dtype, tX, tW, tY, forms, X, W, Y, stream): tt_fc_forward_static
PyObject *forward_static(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    Args g(args, n, 13);
    auto fn = g.address<decltype(&tt_fc_forward_static)>();
    const tt_layer *lay = g.layer();
    const int64_t batch = g.i64();
    const int k = g.i32(), dt = g.dtype();
    const tt_tiling tX = g.tiling(), tW = g.tiling(), tY = g.tiling();
    uint8_t fb[TT_MAX_K];
    void *x[kMaxShards], *w[kMaxShards], *y[kMaxShards];
    const uint8_t *f = g.forms(fb);
    void **X = g.shards(x), **W = g.shards(w), **Y = g.shards(y);
    void *stream = g.stream();
    return finish(g, [&] { return fn(lay, batch, k, dt, tX, tW, tY, f, in(X), in(W), Y, stream); });
}

// backward(address, layer, batch, k, dtype, tX, tW, tY, tdY, tdX, forms_dgrad, forms_wgrad, X, W, Y, dY, dX, dW, workspace,
// stream): tt_fc_backward, tt_conv_backward
PyObject *backward(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    Args g(args, n, 20);
    auto fn = g.address<decltype(&tt_fc_backward)>();
    const tt_layer *lay = g.layer();
    const int64_t batch = g.i64();
    const int k = g.i32(), dt = g.dtype();
    const tt_tiling tX = g.tiling(), tW = g.tiling(), tY = g.tiling(), tdY = g.tiling(), tdX = g.tiling();
    uint8_t fdb[TT_MAX_K], fwb[TT_MAX_K];
    void *x[kMaxShards], *w[kMaxShards], *y[kMaxShards], *dy[kMaxShards], *dx[kMaxShards], *dw[kMaxShards];
    const uint8_t *fd = g.forms(fdb), *fw = g.forms(fwb);
    void **X = g.shards(x), **W = g.shards(w), **Y = g.shards(y), **dY = g.shards(dy), **dX = g.shards(dx), **dW = g.shards(dw);
    size_t bytes;
    void *ws = g.workspace(&bytes), *stream = g.stream();
    return finish(g, [&] {
        return fn(lay, batch, k, dt, tX, tW, tY, tdY, tdX, fd, fw, in(X), in(W), in(Y), in(dY), dX, dW, ws, bytes, stream);
    });
}

// flatten(address, dst, B, src, A, k, batch, channels, pixels, elem_bytes, to_matrix, stream): tt_flatten
PyObject *flatten(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    Args g(args, n, 12);
    auto fn = g.address<decltype(&tt_flatten)>();
    void *d[kMaxShards], *s[kMaxShards];
    void **dst = g.shards(d);
    const tt_tiling B = g.tiling();
    void **src = g.shards(s);
    const tt_tiling A = g.tiling();
    const int k = g.i32();
    const int64_t batch = g.i64(), channels = g.i64(), pixels = g.i64();
    const int eb = g.i32(), to_matrix = g.flag();
    void *stream = g.stream();
    return finish(g, [&] { return fn(dst, B, in(src), A, k, batch, channels, pixels, eb, to_matrix, stream); });
}

// retile(address, dst, B, src, A, k, rows, cols, elem_bytes, stream): tt_retile
PyObject *retile(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    Args g(args, n, 10);
    auto fn = g.address<decltype(&tt_retile)>();
    void *d[kMaxShards], *s[kMaxShards];
    void **dst = g.shards(d);
    const tt_tiling B = g.tiling();
    void **src = g.shards(s);
    const tt_tiling A = g.tiling();
    const int k = g.i32();
    const int64_t rows = g.i64(), cols = g.i64();
    const int eb = g.i32();
    void *stream = g.stream();
    return finish(g, [&] { return fn(dst, B, in(src), A, k, rows, cols, eb, stream); });
}

// converters(tiling, forms, dtype): what the binding uses for arguments that are no plain strings
PyObject *converters(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != 3) {
        PyErr_SetString(PyExc_TypeError, "3 arguments expected");
        return nullptr;
    }
    PyObject **const to[3] = {&g_tiling, &g_forms, &g_dtype};
    for (int i = 0; i < 3; ++i) {
        Py_INCREF(args[i]);
        Py_XSETREF(*to[i], args[i]);
    }
    Py_RETURN_NONE;
}

template <PyObject *(*F)(PyObject *, PyObject *const *, Py_ssize_t)> PyMethodDef method_def(const char *name)
{
    return {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(F)), METH_FASTCALL, nullptr};
}

PyMethodDef g_methods[] = {method_def<forward>("forward"), method_def<forward_static>("forward_static"), method_def<backward>("backward"),
                           method_def<flatten>("flatten"), method_def<retile>("retile"), method_def<converters>("converters"),
                           {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

} // namespace

PyMODINIT_FUNC PyInit__calls()
{
    g_data_ptr = PyUnicode_InternFromString("data_ptr");
    g_numel = PyUnicode_InternFromString("numel");
    g_element_size = PyUnicode_InternFromString("element_size");
    g_value = PyUnicode_InternFromString("value");
    if (!g_data_ptr || !g_numel || !g_element_size || !g_value) return nullptr;
    return PyModule_Create(&g_module);
}
