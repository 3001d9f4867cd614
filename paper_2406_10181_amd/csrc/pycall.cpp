// CPython module `_call`: argument marshalling for the entry points a training program calls in every step.
//
// The binding's general path (ctypes) converts a dozen arguments at about 0.1 us each besides the Python code that
// collects them: 2.2 us for lsp_compress_planned and 2.6 us for lsp_decompress_apply, a fifth of what enqueuing a small
// problem's kernels costs.  Here it is 0.7 and 1.1 us.  Nothing else happens in this file; the functions called are those of the
// C ABI, whose addresses the binding hands over once (bind), so this module links against nothing but Python.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include "lsp.h"

namespace {

PyObject* g_data_ptr;      // interned names
PyObject* g_cuda_stream;
PyObject* g_ctypes;
PyObject* g_data;
PyObject* g_argument_error;   // ctypes.ArgumentError

decltype(&lsp_compress_planned) g_compress_planned;
decltype(&lsp_decompress_apply) g_decompress_apply;
decltype(&lsp_compress_planned_grouped) g_compress_grouped;
decltype(&lsp_decompress_apply_grouped) g_apply_grouped;

// Converts one argument after another, to what ctypes makes of it; the first failure leaves a Python exception and ok = false.
struct Args {
    PyObject* const* first;
    PyObject* const* a = first;
    bool ok = true;

    explicit Args(PyObject* const* args) : first(args) {}
    void refuse() {                                    // the argument before `a`
        PyErr_Format(g_argument_error, "argument %zd: TypeError: wrong type", (Py_ssize_t)(a - first));
        ok = false;
    }
    // the low bits of an integer, however large: a value that makes no sense is the library's to refuse
    uint64_t integer() {
        PyObject* x = *a++;
        if (!ok) return 0;
        const uint64_t v = PyLong_AsUnsignedLongLongMask(x);
        if (v == (uint64_t)-1 && PyErr_Occurred()) { PyErr_Clear(); refuse(); }
        return v;
    }
    int64_t int64() { return (int64_t)integer(); }
    int32_t int32() { return (int32_t)integer(); }
    // address held by a Python int (None: NULL), and gives the reference up
    void* taken(PyObject* i) {
        if (!i) { ok = false; return nullptr; }
        void* p = nullptr;
        if (PyLong_Check(i)) p = reinterpret_cast<void*>((uintptr_t)PyLong_AsUnsignedLongLongMask(i));
        else if (i != Py_None) refuse();
        Py_DECREF(i);
        return p;
    }
    // a tensor, a numpy array, an address or None
    void* pointer() {
        PyObject* x = *a++;
        if (!ok || x == Py_None) return nullptr;
        if (PyLong_Check(x)) { Py_INCREF(x); return taken(x); }
        PyObject* i = PyObject_CallMethodNoArgs(x, g_data_ptr);
        if (!i && PyErr_ExceptionMatches(PyExc_AttributeError)) {
            PyErr_Clear();
            if (PyObject* c = PyObject_GetAttr(x, g_ctypes)) {
                i = PyObject_GetAttr(c, g_data);
                Py_DECREF(c);
            } else if (PyErr_ExceptionMatches(PyExc_AttributeError)) {
                PyErr_Format(PyExc_TypeError, "cannot take the address of %R", (PyObject*)Py_TYPE(x));
            }
        }
        return taken(i);
    }
    // a torch stream, an address or None
    void* stream() {
        PyObject* x = *a++;
        if (!ok || x == Py_None) return nullptr;
        if (PyLong_Check(x)) { Py_INCREF(x); return taken(x); }
        return taken(PyObject_GetAttr(x, g_cuda_stream));
    }
};

bool count_is(Py_ssize_t have, Py_ssize_t want) {
    if (have == want) return true;
    PyErr_Format(PyExc_TypeError, "%zd arguments, %zd expected", have, want);
    return false;
}

template <typename F> PyObject* without_gil(F&& call) {
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = call();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// (G, plan, m, n, r, d, S, dtype, workspace, workspace_bytes, stream)
PyObject* compress_planned(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    if (!count_is(nargs, 11)) return nullptr;
    Args a(args);
    const void* G = a.pointer(); const void* plan = a.pointer();
    const int64_t m = a.int64(), n = a.int64();
    const int32_t r = a.int32(), d = a.int32();
    float* S = static_cast<float*>(a.pointer());
    const int32_t dtype = a.int32();
    void* ws = a.pointer();
    const size_t bytes = a.integer();
    void* st = a.stream();
    if (!a.ok) return nullptr;
    return without_gil([&] { return g_compress_planned(G, plan, m, n, r, d, S, static_cast<lsp_dtype>(dtype), ws, bytes, st); });
}

// (W, S, P_idx, P_val, Q_idx, Q_val, m, n, r, d, dtype, stream)
PyObject* decompress_apply(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    if (!count_is(nargs, 12)) return nullptr;
    Args a(args);
    void* W = a.pointer();
    const float* S = static_cast<const float*>(a.pointer());
    const int32_t* P_idx = static_cast<const int32_t*>(a.pointer());
    const float* P_val = static_cast<const float*>(a.pointer());
    const int32_t* Q_idx = static_cast<const int32_t*>(a.pointer());
    const float* Q_val = static_cast<const float*>(a.pointer());
    const int64_t m = a.int64(), n = a.int64();
    const int32_t r = a.int32(), d = a.int32(), dtype = a.int32();
    void* st = a.stream();
    if (!a.ok) return nullptr;
    return without_gil([&] { return g_decompress_apply(W, S, P_idx, P_val, Q_idx, Q_val, m, n, r, d, static_cast<lsp_dtype>(dtype), st); });
}

// (address of the items, count, r, d, dtype, stream)
template <typename Item, typename Entry> PyObject* grouped(Entry entry, PyObject* const* args, Py_ssize_t nargs) {
    if (!count_is(nargs, 6)) return nullptr;
    Args a(args);
    const Item* items = static_cast<const Item*>(a.pointer());
    const int32_t count = a.int32(), r = a.int32(), d = a.int32(), dtype = a.int32();
    void* st = a.stream();
    if (!a.ok) return nullptr;
    return without_gil([&] { return entry(items, count, r, d, static_cast<lsp_dtype>(dtype), st); });
}
PyObject* compress_planned_grouped(PyObject*, PyObject* const* args, Py_ssize_t nargs) { return grouped<lsp_compress_item>(g_compress_grouped, args, nargs); }
PyObject* decompress_apply_grouped(PyObject*, PyObject* const* args, Py_ssize_t nargs) { return grouped<lsp_apply_item>(g_apply_grouped, args, nargs); }

// (addresses of the four functions, in the order of the methods)
PyObject* bind(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    if (!count_is(nargs, 4)) return nullptr;
    Args a(args);
    void* p[4];
    for (void*& x : p) x = a.pointer();
    if (!a.ok) return nullptr;
    g_compress_planned = reinterpret_cast<decltype(g_compress_planned)>(p[0]);
    g_decompress_apply = reinterpret_cast<decltype(g_decompress_apply)>(p[1]);
    g_compress_grouped = reinterpret_cast<decltype(g_compress_grouped)>(p[2]);
    g_apply_grouped = reinterpret_cast<decltype(g_apply_grouped)>(p[3]);
    Py_RETURN_NONE;
}

template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)> PyMethodDef method(const char* name) {
    return {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(F)), METH_FASTCALL, nullptr};
}
PyMethodDef g_methods[] = {
    method<compress_planned>("compress_planned"), method<decompress_apply>("decompress_apply"),
    method<compress_planned_grouped>("compress_planned_grouped"), method<decompress_apply_grouped>("decompress_apply_grouped"),
    method<bind>("bind"), {nullptr, nullptr, 0, nullptr},
};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_call", "Argument marshalling of the per-step entry points.", -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__call(void) {
    g_data_ptr = PyUnicode_InternFromString("data_ptr");
    g_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    g_ctypes = PyUnicode_InternFromString("ctypes");
    g_data = PyUnicode_InternFromString("data");
    PyObject* ctypes = PyImport_ImportModule("ctypes");
    if (!ctypes) return nullptr;
    g_argument_error = PyObject_GetAttrString(ctypes, "ArgumentError");
    Py_DECREF(ctypes);
    if (!g_argument_error) return nullptr;
    return PyModule_Create(&g_module);
}
