// The calls a serving step makes, attention and append, marshalled in C for binding.py (CPython extension `_calls`).
//
// A call through ctypes spends about 1.4 us on its arguments before the library is entered, a fifth of what a small
// call costs in all (the launch itself takes 2.3 us).  Here it is 0.3 us.  What is handled is what such a program passes:
// the two structs as binding.py makes them, tensors (anything with data_ptr()), integer addresses, None, plain numbers.
// Anything else -- other types, wrong counts or names of arguments, a library that is not loaded yet -- goes to the
// ctypes function of binding.py with the arguments as they came, so that results and errors are its own.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstddef>
#include <cstdint>

namespace {

typedef int (*AttnFn)(const void*, const void*, const void*, const void*, const void*, void*, int32_t, float, uint32_t, void*, size_t, void*);
typedef int (*AppendFn)(const void*, const void*, const void*, const void*, void*);

// Set once per loaded library by bind(), under the GIL.
AttnFn attn_fn = nullptr;
AppendFn append_fn = nullptr;
PyObject *bound_lib = nullptr, *module_dict = nullptr, *lib_name = nullptr, *data_ptr_name = nullptr;
PyObject *pool_type = nullptr, *batch_type = nullptr, *check = nullptr, *slow_attn = nullptr, *slow_append = nullptr;

bool ready() { return bound_lib && PyDict_GetItemWithError(module_dict, lib_name) == bound_lib; }

// false: not one of the plain cases (no Python error is left set)
bool address(PyObject* o, void** out) {
    if (o == Py_None) {
        *out = nullptr;
        return true;
    }
    if (PyLong_CheckExact(o)) {
        *out = reinterpret_cast<void*>(static_cast<uintptr_t>(PyLong_AsUnsignedLongLongMask(o)));
        if (!PyErr_Occurred()) return true;
        PyErr_Clear();
        return false;
    }
    PyObject* r = PyObject_CallMethodNoArgs(o, data_ptr_name);
    const bool ok = r && PyLong_CheckExact(r);
    if (ok) *out = reinterpret_cast<void*>(static_cast<uintptr_t>(PyLong_AsUnsignedLongLongMask(r)));
    Py_XDECREF(r);
    if (PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    return ok;
}

// the caller's argument keeps the struct alive during the call
bool structure(PyObject* o, PyObject* type, void** out) {
    if (reinterpret_cast<PyObject*>(Py_TYPE(o)) != type) return false;
    Py_buffer view;
    if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) {
        PyErr_Clear();
        return false;
    }
    *out = view.buf;
    PyBuffer_Release(&view);
    return true;
}

bool whole(PyObject* o, long long* out) {
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    *out = PyLong_AsLongLongAndOverflow(o, &overflow);
    return overflow == 0 && !PyErr_Occurred();
}

// Arguments by position and name into slots[0, n); false where that does not work out.
bool collect(PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames, const char* const* names, Py_ssize_t n, PyObject** slots) {
    if (nargs > n) return false;
    for (Py_ssize_t i = 0; i < n; ++i) slots[i] = i < nargs ? args[i] : nullptr;
    const Py_ssize_t nkw = kwnames ? PyTuple_GET_SIZE(kwnames) : 0;
    for (Py_ssize_t k = 0; k < nkw; ++k) {
        Py_ssize_t i = nargs;
        while (i < n && PyUnicode_CompareWithASCIIString(PyTuple_GET_ITEM(kwnames, k), names[i]) != 0) ++i;
        if (i == n || slots[i]) return false;
        slots[i] = args[nargs + k];
    }
    return true;
}

PyObject* result(int rc) {
    if (rc >= 0) return PyLong_FromLong(rc);
    return PyObject_CallFunction(check, "i", rc);  // raises with the library's message
}

PyObject* attn(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
    static const char* const names[] = {"pool", "batch", "q", "k_new", "v_new", "out", "q_heads", "softmax_scale", "flags", "workspace",
                                        "workspace_bytes", "stream"};
    PyObject* a[12];
    void *pool, *batch, *q, *k_new, *v_new, *out, *workspace = nullptr, *stream = nullptr;
    long long q_heads, flags = 0, bytes = 0;
    double scale = 0;
    const bool plain = ready() && collect(args, nargs, kwnames, names, 12, a) && a[0] && a[1] && a[2] && a[3] && a[4] && a[5] && a[6] && a[7] &&
                       structure(a[0], pool_type, &pool) && structure(a[1], batch_type, &batch) && address(a[2], &q) && address(a[3], &k_new) &&
                       address(a[4], &v_new) && address(a[5], &out) && whole(a[6], &q_heads) && q_heads >= INT32_MIN && q_heads <= INT32_MAX &&
                       PyFloat_CheckExact(a[7]) && (!a[8] || (whole(a[8], &flags) && flags >= 0 && flags <= UINT32_MAX)) &&
                       (!a[9] || address(a[9], &workspace)) && (!a[10] || (whole(a[10], &bytes) && bytes >= 0)) &&
                       (!a[11] || ((a[11] == Py_None || PyLong_CheckExact(a[11])) && address(a[11], &stream)));
    if (!plain) return PyErr_Occurred() ? nullptr : PyObject_Vectorcall(slow_attn, args, nargs, kwnames);
    scale = PyFloat_AS_DOUBLE(a[7]);
    int rc;
    Py_BEGIN_ALLOW_THREADS rc = attn_fn(pool, batch, q, k_new, v_new, out, (int32_t)q_heads, (float)scale, (uint32_t)flags, workspace, (size_t)bytes, stream);
    Py_END_ALLOW_THREADS return result(rc);
}

PyObject* append(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
    static const char* const names[] = {"pool", "batch", "k_new", "v_new", "stream"};
    PyObject* a[5];
    void *pool, *batch, *k_new, *v_new, *stream = nullptr;
    const bool plain = ready() && collect(args, nargs, kwnames, names, 5, a) && a[0] && a[1] && a[2] && a[3] && structure(a[0], pool_type, &pool) &&
                       structure(a[1], batch_type, &batch) && address(a[2], &k_new) && address(a[3], &v_new) &&
                       (!a[4] || ((a[4] == Py_None || PyLong_CheckExact(a[4])) && address(a[4], &stream)));
    if (!plain) return PyErr_Occurred() ? nullptr : PyObject_Vectorcall(slow_append, args, nargs, kwnames);
    int rc;
    Py_BEGIN_ALLOW_THREADS rc = append_fn(pool, batch, k_new, v_new, stream);
    Py_END_ALLOW_THREADS return result(rc);
}

void keep(PyObject** slot, PyObject* o) {
    Py_INCREF(o);
    Py_XSETREF(*slot, o);
}

// setup(module dict, pool type, batch type, check, ctypes functions): once, when binding.py is imported
PyObject* setup(PyObject*, PyObject* args) {
    PyObject *d, *p, *b, *c, *fa, *fp;
    if (!PyArg_ParseTuple(args, "O!OOOOO", &PyDict_Type, &d, &p, &b, &c, &fa, &fp)) return nullptr;
    keep(&module_dict, d), keep(&pool_type, p), keep(&batch_type, b), keep(&check, c), keep(&slow_attn, fa), keep(&slow_append, fp);
    Py_RETURN_NONE;
}

// bind(library object, addresses of its functions)
PyObject* bind(PyObject*, PyObject* args) {
    PyObject* lib;
    unsigned long long fa, fp;
    if (!PyArg_ParseTuple(args, "OKK", &lib, &fa, &fp)) return nullptr;
    attn_fn = reinterpret_cast<AttnFn>(static_cast<uintptr_t>(fa));
    append_fn = reinterpret_cast<AppendFn>(static_cast<uintptr_t>(fp));
    keep(&bound_lib, lib);
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"ragc_prefill_attn", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(attn)), METH_FASTCALL | METH_KEYWORDS,
     "ragc_prefill_attn(pool, batch, q, k_new, v_new, out, q_heads, softmax_scale, flags=0, workspace=None, workspace_bytes=0, stream=0)\n--\n\n"},
    {"ragc_kv_append", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(append)), METH_FASTCALL | METH_KEYWORDS,
     "ragc_kv_append(pool, batch, k_new, v_new, stream=0)\n--\n\n"},
    {"setup", setup, METH_VARARGS, nullptr},
    {"bind", bind, METH_VARARGS, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls() {
    lib_name = PyUnicode_InternFromString("_lib");
    data_ptr_name = PyUnicode_InternFromString("data_ptr");
    return lib_name && data_ptr_name ? PyModule_Create(&module) : nullptr;
}
