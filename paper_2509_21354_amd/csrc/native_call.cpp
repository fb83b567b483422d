// The marshalling of binding.py's calls, as a CPython module: a call of the C ABI from Python spent 5 us on its arguments (two
// method calls per tensor from bytecode, ctypes' conversions, the current stream through two layers of Python) next to some 2 us
// for the launch itself, which is what a decode step of one layer, whose kernel takes 4 us, or a frame's dozen small calls
// then waited for.  The same steps here take about 1 us.
//
// Each function takes the positional arguments of the Python function of its name, asks tensors for is_contiguous() and
// data_ptr() (as Python code does, so whatever overrides them still does) and calls the library with the GIL released.  It
// returns the status, or None if some argument is not of the plain kind (an exact Shape, a tensor, a RowsFrom, an int that fits,
// None): then, and before torch has initialised the GPU or the library is loaded, binding.py marshals through ctypes, which
// says what is wrong.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <stddef.h>
#include <stdint.h>

#include "../../include/kvev.h"

namespace {

// bound once by binding.py: types, what the current stream is asked of, and the library's entry points
PyObject *g_shape_type, *g_rows_type, *g_tensor_type, *g_initialized, *g_get_device, *g_raw_stream;
PyObject *s_is_contiguous, *s_data_ptr, *s_numel, *s_ptr;

enum Entry { kPool, kGate, kGatePrepared, kSelect, kGated, kDense, kRetain, kCompact, kEntries };
const char *const kNames[kEntries] = {"kvev_chunk_pool", "kvev_lstm_gate", "kvev_lstm_gate_prepared", "kvev_select",
                                      "kvev_gated_attention", "kvev_dense_attention", "kvev_retain", "kvev_compact_attention"};
void *g_entry[kEntries];

// Arguments are read one after the other; the first that is not plain leaves `plain` false, an exception leaves `error` true,
// and either turns the rest into no-ops.
struct Reader {
    PyObject *const *args;
    Py_ssize_t n, at = 0;
    bool plain = true, error = false;
    Py_buffer shape_view{};
    bool has_view = false;

    Reader(PyObject *const *a, Py_ssize_t count, Py_ssize_t want) : args(a), n(count) { plain = g_shape_type && count == want; }
    Reader(const Reader &) = delete;
    ~Reader()
    {
        if (has_view) PyBuffer_Release(&shape_view);
    }
    bool ok() const { return plain && !error; }
    PyObject *next() { return args[at++]; }

    const kvev_shape *shape()
    {
        if (!ok()) return nullptr;
        PyObject *o = next();
        if ((PyObject *)Py_TYPE(o) != g_shape_type) { plain = false; return nullptr; }
        if (PyObject_GetBuffer(o, &shape_view, PyBUF_SIMPLE) != 0) { error = true; return nullptr; }
        has_view = true;
        if ((size_t)shape_view.len < sizeof(kvev_shape)) { plain = false; return nullptr; }
        return static_cast<const kvev_shape *>(shape_view.buf);
    }
    int integer()
    {
        if (!ok()) return 0;
        PyObject *o = next();
        if (!PyLong_Check(o)) { plain = false; return 0; }
        int over = 0;
        const long v = PyLong_AsLongAndOverflow(o, &over);
        if (over || v > INT32_MAX || v < INT32_MIN) { plain = false; return 0; }
        return (int)v;
    }
    float real()
    {
        if (!ok()) return 0.f;
        const double v = PyFloat_AsDouble(next());
        if (v == -1.0 && PyErr_Occurred()) { PyErr_Clear(); plain = false; return 0.f; }
        return (float)v;
    }
    // o.name() as a non-negative integer
    size_t ask(PyObject *o, PyObject *name)
    {
        PyObject *r = PyObject_VectorcallMethod(name, &o, 1 | PY_VECTORCALL_ARGUMENTS_OFFSET, nullptr);
        if (!r) { error = true; return 0; }
        size_t v = 0;
        if (PyLong_Check(r)) {
            v = PyLong_AsSize_t(r);
            if (v == (size_t)-1 && PyErr_Occurred()) { PyErr_Clear(); plain = false; }
        } else {
            plain = false;
        }
        Py_DECREF(r);
        return v;
    }
    void *address(PyObject *o, bool check)
    {
        if (!ok() || o == Py_None) return nullptr;
        if (!PyObject_TypeCheck(o, (PyTypeObject *)g_tensor_type)) {
            if ((PyObject *)Py_TYPE(o) != g_rows_type || !check) { plain = false; return nullptr; }
            PyObject *p = PyObject_GetAttr(o, s_ptr);
            if (!p) { error = true; return nullptr; }
            void *v = PyLong_Check(p) ? (void *)PyLong_AsSize_t(p) : nullptr;
            if (!PyLong_Check(p) || PyErr_Occurred()) { PyErr_Clear(); plain = false; }
            Py_DECREF(p);
            return v;
        }
        if (check) {
            PyObject *c = PyObject_VectorcallMethod(s_is_contiguous, &o, 1 | PY_VECTORCALL_ARGUMENTS_OFFSET, nullptr);
            if (!c) { error = true; return nullptr; }
            const int yes = PyObject_IsTrue(c);
            Py_DECREF(c);
            if (yes < 0) { error = true; return nullptr; }
            if (!yes) {
                PyErr_SetString(PyExc_AssertionError, "kvev takes contiguous tensors");
                error = true;
                return nullptr;
            }
        }
        return (void *)ask(o, s_data_ptr);
    }
    void *tensor() { return ok() ? address(next(), true) : nullptr; }
    // a scratch tensor (or None) and its size
    void *scratch(size_t &bytes)
    {
        bytes = 0;
        if (!ok()) return nullptr;
        PyObject *o = next();
        if (o == Py_None) return nullptr;
        if (!PyObject_TypeCheck(o, (PyTypeObject *)g_tensor_type)) { plain = false; return nullptr; }
        void *p = address(o, true);
        if (ok()) bytes = ask(o, s_numel);
        return p;
    }
    // a tuple of `count` tensors, whose addresses go to consecutive fields of `out` (false: None stood in its place)
    bool weights(const void **out, Py_ssize_t count, bool may_be_none)
    {
        if (!ok()) return false;
        PyObject *o = next();
        if (o == Py_None && may_be_none) return false;
        if (!PyTuple_CheckExact(o) || PyTuple_GET_SIZE(o) != count) { plain = false; return false; }
        for (Py_ssize_t i = 0; i < count; ++i) {
            PyObject *t = PyTuple_GET_ITEM(o, i);
            if (t == Py_None) { plain = false; return false; }
            out[i] = address(t, false);
        }
        return true;
    }
    // torch's current stream
    void *stream()
    {
        if (!ok()) return nullptr;
        PyObject *up = PyObject_CallNoArgs(g_initialized);      // (asked of torch: the flag behind it stays set in a forked child)
        if (!up) { error = true; return nullptr; }
        const bool is_up = up == Py_True;
        Py_DECREF(up);
        if (!is_up) { plain = false; return nullptr; }
        PyObject *dev = PyObject_CallNoArgs(g_get_device);
        if (!dev) { error = true; return nullptr; }
        PyObject *r = PyObject_CallOneArg(g_raw_stream, dev);
        Py_DECREF(dev);
        if (!r) { error = true; return nullptr; }
        void *v = (void *)PyLong_AsSize_t(r);
        if (PyErr_Occurred()) { PyErr_Clear(); plain = false; }
        Py_DECREF(r);
        return v;
    }
    template <class F> PyObject *run(F &&call)
    {
        if (error) return nullptr;
        if (!plain) Py_RETURN_NONE;
        int status;
        Py_BEGIN_ALLOW_THREADS
        status = call();
        Py_END_ALLOW_THREADS
        return PyLong_FromLong(status);
    }
};

template <class F> F entry(Entry e, F) { return reinterpret_cast<F>(g_entry[e]); }
#define ENTRY(e, fn) entry(e, static_cast<decltype(&fn)>(nullptr))

PyObject *chunk_pool(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    Reader r(args, n, 11);
    const kvev_shape *sh = r.shape();
    void *K = r.tensor(), *V = r.tensor();
    const int mode = r.integer();
    kvev_mlp_w wK{}, wV{};
    static_assert(sizeof(kvev_mlp_w) == 4 * sizeof(void *) && sizeof(kvev_lstm_w) == 6 * sizeof(void *), "addresses in a row");
    const bool hasK = r.weights(reinterpret_cast<const void **>(&wK), 4, true), hasV = r.weights(reinterpret_cast<const void **>(&wV), 4, true);
    const int c0 = r.integer(), c1 = r.integer();
    void *Kb = r.tensor(), *Vb = r.tensor();
    size_t bytes;
    void *ws = r.scratch(bytes), *st = r.stream();
    return r.run([&] { return ENTRY(kPool, kvev_chunk_pool)(sh, K, V, mode, hasK ? &wK : nullptr, hasV ? &wV : nullptr, c0, c1, Kb, Vb, ws, bytes, st); });
}

PyObject *lstm_gate(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    Reader r(args, n, 11);
    const kvev_shape *sh = r.shape();
    void *Kb = r.tensor(), *Vb = r.tensor();
    kvev_lstm_w w{};
    r.weights(reinterpret_cast<const void **>(&w), 6, false);
    const int c0 = r.integer(), c1 = r.integer();
    void *h = r.tensor(), *c = r.tensor(), *util = r.tensor(), *gate = r.tensor();
    size_t bytes;
    void *ws = r.scratch(bytes), *st = r.stream();
    return r.run([&] { return ENTRY(kGate, kvev_lstm_gate)(sh, Kb, Vb, &w, c0, c1, (float *)h, (float *)c, (float *)util, (float *)gate, ws, bytes, st); });
}

PyObject *lstm_gate_prepared(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    Reader r(args, n, 12);
    const kvev_shape *sh = r.shape();
    void *Kb = r.tensor(), *Vb = r.tensor();
    kvev_lstm_w w{};
    r.weights(reinterpret_cast<const void **>(&w), 6, false);
    size_t pbytes;
    void *packed = r.scratch(pbytes);
    const int c0 = r.integer(), c1 = r.integer();
    void *h = r.tensor(), *c = r.tensor(), *util = r.tensor(), *gate = r.tensor();
    size_t bytes;
    void *ws = r.scratch(bytes), *st = r.stream();
    return r.run([&] {
        return ENTRY(kGatePrepared, kvev_lstm_gate_prepared)(sh, Kb, Vb, &w, packed, pbytes, c0, c1, (float *)h, (float *)c, (float *)util, (float *)gate, ws, bytes, st);
    });
}

PyObject *select_(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    Reader r(args, n, 9);
    const kvev_shape *sh = r.shape();
    void *util = r.tensor(), *gate = r.tensor();
    const int mode = r.integer(), k = r.integer();
    const float tau = r.real();
    const int k_cap = r.integer();
    void *idx = r.tensor(), *count = r.tensor(), *st = r.stream();
    return r.run([&] { return ENTRY(kSelect, kvev_select)(sh, (float *)util, (float *)gate, mode, k, tau, k_cap, (int32_t *)idx, (int32_t *)count, st); });
}

PyObject *gated_attention(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    Reader r(args, n, 13);
    const kvev_shape *sh = r.shape();
    void *Q = r.tensor();
    const int Tq = r.integer();
    void *K = r.tensor(), *V = r.tensor(), *Kb = r.tensor(), *Vb = r.tensor(), *idx = r.tensor(), *count = r.tensor();
    const int k_cap = r.integer();
    void *O = r.tensor();
    size_t bytes;
    void *ws = r.scratch(bytes);
    const int causal = r.integer();
    void *st = r.stream();
    return r.run([&] { return ENTRY(kGated, kvev_gated_attention)(sh, Q, Tq, K, V, Kb, Vb, (int32_t *)idx, (int32_t *)count, k_cap, causal, O, ws, bytes, st); });
}

PyObject *dense_attention(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    Reader r(args, n, 8);
    const kvev_shape *sh = r.shape();
    void *Q = r.tensor();
    const int Tq = r.integer();
    void *K = r.tensor(), *V = r.tensor(), *O = r.tensor();
    size_t bytes;
    void *ws = r.scratch(bytes);
    const int causal = r.integer();
    void *st = r.stream();
    return r.run([&] { return ENTRY(kDense, kvev_dense_attention)(sh, Q, Tq, K, V, causal, O, ws, bytes, st); });
}

PyObject *retain(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    Reader r(args, n, 14);
    const kvev_shape *sh = r.shape();
    const int k = r.integer(), k_cap = r.integer();
    void *Kn = r.tensor(), *Vn = r.tensor(), *un = r.tensor();
    const int cap = r.integer(), first = r.integer(), m = r.integer();
    void *Kc = r.tensor(), *Vc = r.tensor(), *ids = r.tensor(), *uc = r.tensor(), *count = r.tensor(), *st = r.stream();
    return r.run([&] {
        return ENTRY(kRetain, kvev_retain)(sh, k, k_cap, Kn, Vn, (float *)un, cap, first, m, Kc, Vc, (int32_t *)ids, (float *)uc, (int32_t *)count, st);
    });
}

PyObject *compact_attention(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    Reader r(args, n, 13);
    const kvev_shape *sh = r.shape();
    void *Q = r.tensor();
    const int Tq = r.integer();
    void *Kw = r.tensor(), *Vw = r.tensor(), *Kc = r.tensor(), *Vc = r.tensor(), *count = r.tensor();
    const int k_cap = r.integer();
    void *O = r.tensor();
    size_t bytes;
    void *ws = r.scratch(bytes);
    const int causal = r.integer(), first = r.integer();
    void *st = r.stream();
    return r.run([&] { return ENTRY(kCompact, kvev_compact_attention)(sh, Q, Tq, Kw, Vw, first, Kc, Vc, (int32_t *)count, k_cap, causal, O, ws, bytes, st); });
}

// bind(Shape, RowsFrom, Tensor, is_initialized, get_device, raw_stream, {name: address})
PyObject *bind(PyObject *, PyObject *args)
{
    PyObject *shape, *rows, *tensor, *up, *dev, *raw, *entries;
    if (!PyArg_ParseTuple(args, "O!O!O!OOOO!", &PyType_Type, &shape, &PyType_Type, &rows, &PyType_Type, &tensor, &up, &dev, &raw, &PyDict_Type, &entries))
        return nullptr;
    void *found[kEntries];
    for (int e = 0; e < kEntries; ++e) {
        PyObject *a = PyDict_GetItemString(entries, kNames[e]);
        if (!a) return PyErr_Format(PyExc_KeyError, "%s", kNames[e]);
        found[e] = PyLong_AsVoidPtr(a);
        if (PyErr_Occurred()) return nullptr;
    }
    for (int e = 0; e < kEntries; ++e) g_entry[e] = found[e];
    Py_INCREF(rows); Py_INCREF(tensor); Py_INCREF(up); Py_INCREF(dev); Py_INCREF(raw); Py_INCREF(shape);
    g_rows_type = rows; g_tensor_type = tensor; g_initialized = up; g_get_device = dev; g_raw_stream = raw;
    g_shape_type = shape;           // (the last one: its presence says that all are there)
    Py_RETURN_NONE;
}

#define FAST(name, fn) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(fn)), METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {
    FAST("chunk_pool", chunk_pool), FAST("lstm_gate", lstm_gate), FAST("lstm_gate_prepared", lstm_gate_prepared), FAST("select", select_),
    FAST("gated_attention", gated_attention), FAST("dense_attention", dense_attention), FAST("retain", retain),
    FAST("compact_attention", compact_attention), {"bind", bind, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_native", "Marshalling of calls into libkvev.so.", -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void)
{
    s_is_contiguous = PyUnicode_InternFromString("is_contiguous");
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_numel = PyUnicode_InternFromString("numel");
    s_ptr = PyUnicode_InternFromString("ptr");
    if (!s_is_contiguous || !s_data_ptr || !s_numel || !s_ptr) return nullptr;
    return PyModule_Create(&g_module);
}
