// Python module `_native`: the product and transpose calls of the C ABI for a Python program, without
// ctypes.  A small product takes 3 to 5 us on the device; marshalling its ten arguments in Python
// (int(), data_ptr(), current_stream(), ctypes conversions) took longer than the product itself, so
// the host set the pace: da_spmm on a 4096-row matrix with N = 8 ran at 7.8 us a call.  Here a call is
// one C function that unpacks the arguments in place; everything else (checks, geometry, launch) is
// behind the C ABI as before.  No device code.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <exception>

#include "da_spmm.h"

namespace {

PyObject* g_error = nullptr;          // binding.DaSpmmError
PyObject* g_current_stream = nullptr; // torch.cuda.current_stream, which also initialises the runtime

// Arguments of a call by position or keyword, in the order of `names`; missing ones stay null.
bool collect(const char* fn, const char* const* names, int n, int required, PyObject* const* args, Py_ssize_t nargs,
             PyObject* kwnames, PyObject** out) {
    for (int i = 0; i < n; ++i) out[i] = nullptr;
    if (nargs > n) {
        PyErr_Format(PyExc_TypeError, "%s() takes at most %d arguments (%zd given)", fn, n, nargs);
        return false;
    }
    for (Py_ssize_t i = 0; i < nargs; ++i) out[i] = args[i];
    const Py_ssize_t nkw = kwnames ? PyTuple_GET_SIZE(kwnames) : 0;
    for (Py_ssize_t k = 0; k < nkw; ++k) {
        PyObject* name = PyTuple_GET_ITEM(kwnames, k);
        int i = 0;
        while (i < n && PyUnicode_CompareWithASCIIString(name, names[i]) != 0) ++i;
        if (i == n || out[i]) {
            PyErr_Format(PyExc_TypeError, i == n ? "%s() got an unexpected keyword argument '%U'"
                                                 : "%s() got multiple values for argument '%U'", fn, name);
            return false;
        }
        out[i] = args[nargs + k];
    }
    for (int i = 0; i < required; ++i)
        if (!out[i]) {
            PyErr_Format(PyExc_TypeError, "%s() missing required argument '%s'", fn, names[i]);
            return false;
        }
    return true;
}

bool to_int(PyObject* x, int64_t* out) {
    if (PyLong_CheckExact(x)) {
        *out = (int64_t)PyLong_AsUnsignedLongLongMask(x);
        return !(*out == -1 && PyErr_Occurred());
    }
    PyObject* v = PyNumber_Long(x);
    if (!v) return false;
    *out = (int64_t)PyLong_AsUnsignedLongLongMask(v);
    Py_DECREF(v);
    return !(*out == -1 && PyErr_Occurred());
}

// the value of an attribute (called first when `call`) as an address
bool attribute_address(PyObject* x, const char* name, bool call, void** out) {
    PyObject* v = PyObject_GetAttrString(x, name);
    if (v && call) {
        PyObject* r = PyObject_CallNoArgs(v);
        Py_DECREF(v);
        v = r;
    }
    if (!v) return false;
    *out = PyLong_AsVoidPtr(v);
    Py_DECREF(v);
    return !(!*out && PyErr_Occurred());
}

// device address of a tensor; an int or None passes through
bool to_address(PyObject* x, void** out) {
    if (x == Py_None) { *out = nullptr; return true; }
    if (THPVariable_Check(x)) {
        *out = const_cast<void*>(THPVariable_Unpack(x).const_data_ptr());
        return true;
    }
    if (PyLong_Check(x)) { *out = PyLong_AsVoidPtr(x); return !(!*out && PyErr_Occurred()); }
    return attribute_address(x, "data_ptr", true, out);
}

bool to_stream(PyObject* x, void** out) {
    if (!x || x == Py_None) {
        static bool initialised = false;
        if (!initialised) {                                  // first use: let torch start the runtime (or refuse)
            PyObject* s = PyObject_CallNoArgs(g_current_stream);
            if (!s) return false;
            Py_DECREF(s);
            initialised = true;
        }
        *out = c10::hip::getCurrentHIPStream().stream();
        return true;
    }
    if (PyLong_Check(x)) { *out = PyLong_AsVoidPtr(x); return !(!*out && PyErr_Occurred()); }
    return attribute_address(x, "cuda_stream", false, out);
}

PyObject* finish(int status) {
    if (status == DA_OK) Py_RETURN_NONE;
    PyObject* e = PyObject_CallFunction(g_error, "is", status, da_spmm_last_error());
    if (e) {
        PyErr_SetObject(g_error, e);
        Py_DECREF(e);
    }
    return nullptr;
}

template <class F>
PyObject* guarded(F&& f) {
    try {
        return f();
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

template <class F>
int without_gil(F&& f) {
    PyThreadState* ts = PyEval_SaveThread();
    const int st = f();
    PyEval_RestoreThread(ts);
    return st;
}

PyObject* py_spmm(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
    static const char* const names[] = {"m", "k", "N", "rowptr", "colind", "vals", "B", "C", "algo", "stream"};
    return guarded([&]() -> PyObject* {
        PyObject* a[10];
        int64_t n[3], algo;
        void *p[5], *stream;
        if (!collect("da_spmm", names, 10, 9, args, nargs, kwnames, a)) return nullptr;
        for (int i = 0; i < 3; ++i) if (!to_int(a[i], &n[i])) return nullptr;
        for (int i = 0; i < 5; ++i) if (!to_address(a[3 + i], &p[i])) return nullptr;
        if (!to_int(a[8], &algo) || !to_stream(a[9], &stream)) return nullptr;
        return finish(without_gil([&] {
            return da_spmm(n[0], n[1], n[2], (const int32_t*)p[0], (const int32_t*)p[1], (const float*)p[2],
                           (const float*)p[3], (float*)p[4], (int)algo, stream);
        }));
    });
}

PyObject* py_spmm_ex(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
    static const char* const names[] = {"m", "k", "N", "rowptr", "colind", "vals", "B", "ldb", "layout_b", "C", "ldc",
                                        "layout_c", "algo", "stream"};
    return guarded([&]() -> PyObject* {
        PyObject* a[14];
        int64_t n[3], ldb, lb, ldc, lc, algo;
        void *p[4], *c, *stream;
        if (!collect("da_spmm_ex", names, 14, 13, args, nargs, kwnames, a)) return nullptr;
        for (int i = 0; i < 3; ++i) if (!to_int(a[i], &n[i])) return nullptr;
        for (int i = 0; i < 4; ++i) if (!to_address(a[3 + i], &p[i])) return nullptr;
        if (!to_int(a[7], &ldb) || !to_int(a[8], &lb) || !to_address(a[9], &c) || !to_int(a[10], &ldc) ||
            !to_int(a[11], &lc) || !to_int(a[12], &algo) || !to_stream(a[13], &stream)) return nullptr;
        return finish(without_gil([&] {
            return da_spmm_ex(n[0], n[1], n[2], (const int32_t*)p[0], (const int32_t*)p[1], (const float*)p[2],
                              (const float*)p[3], ldb, (int)lb, (float*)c, ldc, (int)lc, (int)algo, stream);
        }));
    });
}

PyObject* py_transpose(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
    static const char* const names[] = {"m", "k", "nnz", "rowptr", "colind", "vals", "t_rowptr", "t_colind", "t_vals",
                                        "workspace", "workspace_bytes", "stream"};
    return guarded([&]() -> PyObject* {
        PyObject* a[12];
        int64_t n[3], bytes;
        void *p[7], *stream;
        if (!collect("da_csr_transpose", names, 12, 11, args, nargs, kwnames, a)) return nullptr;
        for (int i = 0; i < 3; ++i) if (!to_int(a[i], &n[i])) return nullptr;
        for (int i = 0; i < 7; ++i) if (!to_address(a[3 + i], &p[i])) return nullptr;
        if (!to_int(a[10], &bytes) || !to_stream(a[11], &stream)) return nullptr;
        return finish(without_gil([&] {
            return da_csr_transpose(n[0], n[1], n[2], (const int32_t*)p[0], (const int32_t*)p[1], (const float*)p[2],
                                    (int32_t*)p[3], (int32_t*)p[4], (float*)p[5], p[6], (size_t)bytes, stream);
        }));
    });
}

// setup(error class, function that returns the current stream)
PyObject* py_setup(PyObject*, PyObject* args) {
    PyObject *error, *stream;
    if (!PyArg_ParseTuple(args, "OO", &error, &stream)) return nullptr;
    Py_INCREF(error);
    Py_INCREF(stream);
    Py_XSETREF(g_error, error);
    Py_XSETREF(g_current_stream, stream);
    Py_RETURN_NONE;
}

PyMethodDef kMethods[] = {
    {"setup", py_setup, METH_VARARGS, nullptr},
    {"da_spmm", (PyCFunction)(void (*)(void))py_spmm, METH_FASTCALL | METH_KEYWORDS,
     "da_spmm(m, k, N, rowptr, colind, vals, B, C, algo, stream=None)\n--\n\n"
     "C = A.B on the device; arguments as in include/da_spmm.h (torch CUDA tensors or addresses)."},
    {"da_spmm_ex", (PyCFunction)(void (*)(void))py_spmm_ex, METH_FASTCALL | METH_KEYWORDS,
     "da_spmm_ex(m, k, N, rowptr, colind, vals, B, ldb, layout_b, C, ldc, layout_c, algo, stream=None)\n--\n\n"
     "C = A.B with explicit storage order (DA_ROW_MAJOR / DA_COL_MAJOR) and leading dimensions."},
    {"da_csr_transpose", (PyCFunction)(void (*)(void))py_transpose, METH_FASTCALL | METH_KEYWORDS,
     "da_csr_transpose(m, k, nnz, rowptr, colind, vals, t_rowptr, t_colind, t_vals, workspace, workspace_bytes, "
     "stream=None)\n--\n\n"
     "CSR arrays of A^T on the device; arguments as in include/da_spmm.h."},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_native", "Calls of the da_spmm C ABI without ctypes.", -1, kMethods,
                       nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&kModule); }
