// CPython side of the binding: turns the arguments of the calls that a program makes per pass
// (tensors, lists of them, ConvDesc structures, streams) into the C ABI's pointers and calls it.
// Argument marshalling only; the same entry points as include/nnv.h.
//
// Why it is compiled: a batch-1 layer runs for 3-4 us, and marshalling through ctypes took longer
// than that (one nnv_conv_forward call 7.5 us on the host against 3.8 us on the GPU, a forward call
// over 52 layers 53 us).  A pointer costs one data_ptr() method call here, a descriptor one copy of its 52
// bytes, the current stream two calls into torch's own bindings.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <cstring>
#include <vector>
#include "nnv.h"

namespace {

PyObject *g_desc_type, *g_fail, *g_slow_stream, *g_get_device, *g_raw_stream;    // handed over by setup()
PyObject *g_data_ptr, *g_numel, *g_element_size, *g_cuda_stream;                 // interned names
bool g_stream_ready = false;     // torch has initialised the device: the raw calls may be used

bool as_pointer(PyObject *o, void **out) {
    PyObject *v = PyLong_Check(o) ? (Py_INCREF(o), o) : PyObject_CallMethodNoArgs(o, g_data_ptr);
    if (!v) return false;
    *out = PyLong_AsVoidPtr(v);
    Py_DECREF(v);
    return !(*out == nullptr && PyErr_Occurred());
}
bool as_pointer_or_null(PyObject *o, void **out) {
    if (o != Py_None) return as_pointer(o, out);
    *out = nullptr;
    return true;
}

bool as_desc(PyObject *o, nnv_conv_desc *out) {
    if (!PyObject_TypeCheck(o, reinterpret_cast<PyTypeObject *>(g_desc_type))) {
        PyErr_Format(PyExc_TypeError, "expected ConvDesc, got %.100s", Py_TYPE(o)->tp_name);
        return false;
    }
    Py_buffer view;
    if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE)) return false;
    memcpy(out, view.buf, sizeof(*out));
    PyBuffer_Release(&view);
    return true;
}

bool as_kind(PyObject *o, nnv_kind *out) {
    const long v = PyLong_AsLong(o);
    if (v == -1 && PyErr_Occurred()) return false;
    *out = static_cast<nnv_kind>(static_cast<int>(v));
    return true;
}

// An explicit byte count, or the size of the workspace tensor.
bool as_bytes(PyObject *count, PyObject *workspace, size_t *out) {
    *out = 0;
    if (count != Py_None) {
        *out = PyLong_AsSize_t(count);
        return !PyErr_Occurred();
    }
    if (workspace == Py_None) return true;
    PyObject *n = PyObject_CallMethodNoArgs(workspace, g_numel);
    PyObject *e = n ? PyObject_CallMethodNoArgs(workspace, g_element_size) : nullptr;
    if (e) *out = PyLong_AsSize_t(n) * PyLong_AsSize_t(e);
    Py_XDECREF(n);
    Py_XDECREF(e);
    return !PyErr_Occurred();
}

bool as_stream(PyObject *o, void **out) {
    if (o == Py_None) {
        PyObject *v = nullptr;
        if (g_stream_ready && g_raw_stream != Py_None) {
            PyObject *dev = PyObject_CallNoArgs(g_get_device);
            if (dev) v = PyObject_CallOneArg(g_raw_stream, dev);
            Py_XDECREF(dev);
        } else {
            v = PyObject_CallNoArgs(g_slow_stream);      // initialises the device on first use
            g_stream_ready = v != nullptr;
        }
        if (!v) return false;
        *out = PyLong_AsVoidPtr(v);
        Py_DECREF(v);
        return !PyErr_Occurred();
    }
    if (!PyLong_Check(o)) {
        PyObject *v = PyObject_GetAttr(o, g_cuda_stream);
        if (!v) return false;
        *out = PyLong_AsVoidPtr(v);
        Py_DECREF(v);
        return !PyErr_Occurred();
    }
    *out = PyLong_AsVoidPtr(o);
    return !PyErr_Occurred();
}

// A sequence of n items (n < 0: any number, returned through n) as a fast sequence, or null with an error set.
PyObject *as_items(PyObject *o, Py_ssize_t *n) {
    PyObject *s = PySequence_Fast(o, "a list or tuple is wanted");
    if (!s) return nullptr;
    const Py_ssize_t len = PySequence_Fast_GET_SIZE(s);
    if (*n >= 0 && len != *n) {
        Py_DECREF(s);
        PyErr_Format(PyExc_ValueError, "%zd descriptors, but a list of %zd", *n, len);
        return nullptr;
    }
    *n = len;
    return s;
}

template <typename T, typename F>
bool as_array(PyObject *o, Py_ssize_t *n, std::vector<T> *out, F convert) {
    PyObject *s = as_items(o, n);
    if (!s) return false;
    out->resize(*n);
    bool ok = true;
    for (Py_ssize_t i = 0; i < *n && ok; ++i) ok = convert(PySequence_Fast_GET_ITEM(s, i), &(*out)[i]);
    Py_DECREF(s);
    return ok;
}

// None for success, else whatever the Python side raises for the status.
PyObject *finish(int rc, const char *where) {
    if (rc >= 0) Py_RETURN_NONE;
    return PyObject_CallFunction(g_fail, "is", rc, where);
}

bool count_is(Py_ssize_t got, Py_ssize_t want) {
    if (got == want) return true;
    PyErr_Format(PyExc_TypeError, "%zd arguments, %zd are wanted", got, want);
    return false;
}

typedef int (*ForwardFn)(const nnv_conv_desc *, nnv_kind, const void *, const void *, const float *, void *, void *, size_t, void *);

// (desc, kind, x, w_tx, bias, y, workspace, workspace_bytes, stream)
PyObject *forward_with(ForwardFn fn, const char *where, PyObject *const *a, Py_ssize_t n) {
    nnv_conv_desc d;
    nnv_kind kind;
    void *x, *w, *b, *y, *ws, *st;
    size_t bytes;
    if (!count_is(n, 9) || !as_desc(a[0], &d) || !as_kind(a[1], &kind) || !as_pointer_or_null(a[2], &x) ||
        !as_pointer_or_null(a[3], &w) || !as_pointer_or_null(a[4], &b) || !as_pointer_or_null(a[5], &y) ||
        !as_pointer_or_null(a[6], &ws) || !as_bytes(a[7], a[6], &bytes) || !as_stream(a[8], &st))
        return nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = fn(&d, kind, x, w, static_cast<const float *>(b), y, ws, bytes, st);
    Py_END_ALLOW_THREADS
    return finish(rc, where);
}
PyObject *conv_forward(PyObject *, PyObject *const *a, Py_ssize_t n) { return forward_with(nnv_conv_forward, "nnv_conv_forward", a, n); }
PyObject *conv_forward_relu(PyObject *, PyObject *const *a, Py_ssize_t n) { return forward_with(nnv_conv_forward_relu, "nnv_conv_forward_relu", a, n); }

// (desc, kind, x, w_tx, bias, y, stream)
PyObject *conv_forward_static(PyObject *, PyObject *const *a, Py_ssize_t n) {
    nnv_conv_desc d;
    nnv_kind kind;
    void *x, *w, *b, *y, *st;
    if (!count_is(n, 7) || !as_desc(a[0], &d) || !as_kind(a[1], &kind) || !as_pointer_or_null(a[2], &x) ||
        !as_pointer_or_null(a[3], &w) || !as_pointer_or_null(a[4], &b) || !as_pointer_or_null(a[5], &y) || !as_stream(a[6], &st))
        return nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = nnv_conv_forward_static(&d, kind, x, w, static_cast<const float *>(b), y, st);
    Py_END_ALLOW_THREADS
    return finish(rc, "nnv_conv_forward_static");
}

// (desc, kind, w_raw, w_tx, stream)
PyObject *transform_weights(PyObject *, PyObject *const *a, Py_ssize_t n) {
    nnv_conv_desc d;
    nnv_kind kind;
    void *raw, *tx, *st;
    if (!count_is(n, 5) || !as_desc(a[0], &d) || !as_kind(a[1], &kind) || !as_pointer_or_null(a[2], &raw) ||
        !as_pointer_or_null(a[3], &tx) || !as_stream(a[4], &st))
        return nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = nnv_transform_weights(&d, kind, static_cast<const float *>(raw), tx, st);
    Py_END_ALLOW_THREADS
    return finish(rc, "nnv_transform_weights");
}

// (descs, kinds, w_raw, w_tx, stream)
PyObject *transform_weights_grouped(PyObject *, PyObject *const *a, Py_ssize_t n) {
    Py_ssize_t m = -1;
    std::vector<nnv_conv_desc> d;
    std::vector<nnv_kind> kinds;
    std::vector<void *> raw, tx;
    void *st;
    if (!count_is(n, 5) || !as_array(a[0], &m, &d, as_desc) || !as_array(a[1], &m, &kinds, as_kind) ||
        !as_array(a[2], &m, &raw, as_pointer) || !as_array(a[3], &m, &tx, as_pointer) || !as_stream(a[4], &st))
        return nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = nnv_transform_weights_grouped(static_cast<int>(m), d.data(), kinds.data(), reinterpret_cast<const float *const *>(raw.data()), tx.data(), st);
    Py_END_ALLOW_THREADS
    return finish(rc, "nnv_transform_weights_grouped");
}

// (descs, kinds, x, w_tx, bias, y, workspace, workspace_bytes, flags, stream)
PyObject *conv_forward_grouped(PyObject *, PyObject *const *a, Py_ssize_t n) {
    Py_ssize_t m = -1;
    std::vector<nnv_conv_desc> d;
    std::vector<nnv_kind> kinds;
    std::vector<void *> x, w, b, y;
    void *ws, *st;
    size_t bytes;
    if (!count_is(n, 10) || !as_array(a[0], &m, &d, as_desc) || !as_array(a[1], &m, &kinds, as_kind) ||
        !as_array(a[2], &m, &x, as_pointer_or_null) || !as_array(a[3], &m, &w, as_pointer_or_null) ||
        (a[4] != Py_None && !as_array(a[4], &m, &b, as_pointer_or_null)) || !as_array(a[5], &m, &y, as_pointer_or_null) ||
        !as_pointer_or_null(a[6], &ws) || !as_bytes(a[7], a[6], &bytes))
        return nullptr;
    const unsigned long flags = PyLong_AsUnsignedLong(a[8]);
    if (PyErr_Occurred() || !as_stream(a[9], &st)) return nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = nnv_conv_forward_grouped(static_cast<int>(m), d.data(), kinds.data(), x.data(), w.data(),
                                  a[4] == Py_None ? nullptr : reinterpret_cast<const float *const *>(b.data()), y.data(), ws,
                                  bytes, static_cast<unsigned>(flags), st);
    Py_END_ALLOW_THREADS
    return finish(rc, "nnv_conv_forward_grouped");
}

// (descs, kinds, w_raw, w_tx, x, y, workspace, stage_layers, stream_exec, stream_tx); stream_tx None: stream_exec
PyObject *cold_stack(PyObject *, PyObject *const *a, Py_ssize_t n) {
    Py_ssize_t m = -1;
    std::vector<nnv_conv_desc> d;
    std::vector<nnv_kind> kinds;
    std::vector<void *> raw, tx, x, y;
    void *ws, *se, *stx;
    size_t bytes;
    if (!count_is(n, 10) || !as_array(a[0], &m, &d, as_desc) || !as_array(a[1], &m, &kinds, as_kind) ||
        !as_array(a[2], &m, &raw, as_pointer) || !as_array(a[3], &m, &tx, as_pointer) || !as_array(a[4], &m, &x, as_pointer) ||
        !as_array(a[5], &m, &y, as_pointer) || !as_pointer_or_null(a[6], &ws) || !as_bytes(Py_None, a[6], &bytes))
        return nullptr;
    const long stage = PyLong_AsLong(a[7]);
    if (PyErr_Occurred() || !as_stream(a[8], &se)) return nullptr;
    if (a[9] == Py_None) stx = se;
    else if (!as_stream(a[9], &stx)) return nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = nnv_cold_stack(static_cast<int>(m), d.data(), kinds.data(), reinterpret_cast<const float *const *>(raw.data()), tx.data(),
                        x.data(), y.data(), ws, bytes, static_cast<int>(stage), se, stx);
    Py_END_ALLOW_THREADS
    return finish(rc, "nnv_cold_stack");
}

// (ConvDesc type, fail(status, where), current stream handle by torch's public call, current device, raw stream of a device or None)
PyObject *setup(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (!count_is(n, 5)) return nullptr;
    PyObject **slots[5] = {&g_desc_type, &g_fail, &g_slow_stream, &g_get_device, &g_raw_stream};
    if (!PyType_Check(a[0])) {
        PyErr_SetString(PyExc_TypeError, "the first argument is the descriptor type");
        return nullptr;
    }
    for (int i = 0; i < 5; ++i) {
        Py_INCREF(a[i]);
        Py_XSETREF(*slots[i], a[i]);
    }
    Py_RETURN_NONE;
}

#define NNV_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {NNV_METHOD(setup), NNV_METHOD(conv_forward), NNV_METHOD(conv_forward_relu), NNV_METHOD(conv_forward_static),
                           NNV_METHOD(conv_forward_grouped), NNV_METHOD(transform_weights), NNV_METHOD(transform_weights_grouped),
                           NNV_METHOD(cold_stack), {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_nnvpy", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__nnvpy(void) {
    g_data_ptr = PyUnicode_InternFromString("data_ptr");
    g_numel = PyUnicode_InternFromString("numel");
    g_element_size = PyUnicode_InternFromString("element_size");
    g_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    if (!g_data_ptr || !g_numel || !g_element_size || !g_cuda_stream) return nullptr;
    return PyModule_Create(&g_module);
}
