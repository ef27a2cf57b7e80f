// Python module `_native`: what a Python program does for every call, in C++.
//
// (1) The product and transpose calls of the C ABI without ctypes.  A small product takes 3 to 5 us on the
// device; marshalling its ten arguments in Python (int(), data_ptr(), current_stream(), ctypes
// conversions) took longer than the product itself, so the host set the pace: da_spmm on a 4096-row matrix
// with N = 8 ran at 7.8 us a call.
//
// (2) Graphs and graph-convolution layers (gcn.py holds their Python side): the matrix with what is known
// of it, the aggregation A . X with gradient A^T . dY, and the layer relu(A . (X . W) + b), each forward
// and backward one C++ function with one autograd node.  On graphs of a few thousand nodes the device
// needs 20 to 60 us for a layer; separate operations, each with its own Python call and node, took 80 to
// 190 us of host time.
//
// No device code here; all work goes through the C ABI (and, for large dense products, the GEMM library).
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/autocast_mode.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/core/DeviceGuard.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/function.h>
#include <torch/csrc/autograd/functions/utils.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/autograd/saved_variable.h>
#include <torch/csrc/jit/frontend/tracer.h>
#include <torch/csrc/utils/pybind.h>
#include <hip/hip_runtime.h>

#include <atomic>
#include <exception>
#include <memory>
#include <mutex>
#include <optional>
#include <stdexcept>
#include <utility>
#include <vector>

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

// Device address of a tensor, the one its data_ptr() gives: memory that it shares as a lazy copy becomes its
// own first, so that an output is never written into the tensor it was copied from.  A subclass answers for
// itself; an int or None passes through.
bool to_address(PyObject* x, void** out) {
    if (x == Py_None) { *out = nullptr; return true; }
    if (THPVariable_CheckExact(x)) {
        *out = THPVariable_Unpack(x).mutable_data_ptr();
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

// ------------------------------------------------------------------------------------------
// graphs
// ------------------------------------------------------------------------------------------
using at::Tensor;

// A failed call of the C ABI, to be raised as binding.DaSpmmError
struct DaError : std::exception {
    int status;
    std::string text;
    explicit DaError(int st) : status(st), text(da_spmm_last_error()) {}
    const char* what() const noexcept override { return text.c_str(); }
};

void check(int status) {
    if (status != DA_OK) throw DaError(status);
}

void set_error(const DaError& e) {                // the interpreter lock is held
    const py::object err = py::reinterpret_borrow<py::object>(g_error)(e.status, e.text);
    PyErr_SetObject(g_error, err.ptr());
}

// Runs a step of a backward pass.  The autograd engine hands Python exceptions on and makes a plain RuntimeError of
// all others, so errors become Python exceptions here.
template <class F>
auto in_backward(F&& f) {
    auto raise = [](const auto& set) {
        py::gil_scoped_acquire gil;
        set();
        python_error err;
        err.persist();
        throw err;
    };
    try {
        return f();
    } catch (const DaError& e) {
        raise([&] { set_error(e); });
    } catch (const py::builtin_exception& e) {
        raise([&] { e.set_error(); });
    }
    throw std::logic_error("not reached");
}

void* stream_of(const Tensor& t) { return c10::hip::getCurrentHIPStream(t.device().index()).stream(); }

bool capturing(const Tensor& t) {
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    const hipError_t e = hipStreamIsCapturing((hipStream_t)stream_of(t), &status);
    if (e != hipSuccess) (void)hipGetLastError();            // the default stream beside another one's capture
    return e != hipSuccess || status != hipStreamCaptureStatusNone;
}

template <class T> T* data(const Tensor& t) { return t.defined() ? static_cast<T*>(t.data_ptr()) : nullptr; }

// Distance between the rows of a contiguous matrix or of one with unit column stride.  A matrix of one row may
// have any row stride there (a transposed column, an expanded sum): its width does.
int64_t leading(const Tensor& t) { return t.size(0) > 1 ? t.stride(0) : t.size(1); }

// Distance between the rows of a dense operand that this module lays out itself.  A row that is not whole
// 64-byte pieces touches one cache line more on average: with N = 41 a gathered row of B costs 2.3 lines of
// 128 bytes at a distance of 41 and 2 at 48 (power-law graph of 262 144 nodes: 245 and 219 us).
int64_t row_pitch(int64_t n) {
    if (n <= 4) return n;
    if (n <= 8) return 8;
    return (n + 15) / 16 * 16;
}

// The matrix of a graph.  Python may replace its fields while another thread's product runs without the
// interpreter lock, so a graph holds them behind a pointer: a call reads one state of all fields and keeps its
// arrays alive, a change makes a new state.
struct Arrays {
    int64_t m, k, nnz;
    Tensor rowptr, colind, vals;
};
using ArraysPtr = std::shared_ptr<const Arrays>;

struct Graph : std::enable_shared_from_this<Graph> {
    std::mutex arrays_mu;                     // held for a copy of the pointer only
    ArraysPtr arrays;
    std::atomic<bool> prepared{false};
    std::recursive_mutex mu;                  // what follows is filled in by the first calls that need it
    bool have_features = false;
    int eb_products = 0;
    da_features features{};
    std::vector<std::pair<int64_t, int>> algo;
    std::shared_ptr<Graph> t;
    std::weak_ptr<Graph> t_of;

    Graph(int64_t m, int64_t k, const Tensor& rp, const Tensor& ci, const Tensor& va)
        : arrays(std::make_shared<Arrays>(Arrays{m, k, ci.numel(), rp.contiguous(), ci.contiguous(), va.contiguous()})) {}
    ~Graph() {
        if (prepared) da_spmm_release(data<int32_t>(arrays->rowptr));
    }

    ArraysPtr now() {
        std::lock_guard<std::mutex> lk(arrays_mu);
        return arrays;
    }

    template <class T> void change(T Arrays::*field, const T& value) {
        ArraysPtr old;                        // freed after the lock
        std::lock_guard<std::mutex> lk(arrays_mu);
        auto next = std::make_shared<Arrays>(*arrays);
        (*next).*field = value;
        old = std::exchange(arrays, std::move(next));
    }

    const da_features& known() {
        std::lock_guard<std::recursive_mutex> lk(mu);
        if (!have_features) {                 // one device reduction per graph
            const ArraysPtr a = now();
            c10::DeviceGuard guard(a->rowptr.device());
            check(da_spmm_features(a->m, 1, data<int32_t>(a->rowptr), stream_of(a->rowptr), &features));
            have_features = true;
        }
        return features;
    }

    int algo_for(int64_t N) {
        std::lock_guard<std::recursive_mutex> lk(mu);
        for (const auto& a : algo)
            if (a.first == N) return a.second;
        da_features f = known();
        f.N = N;
        const int id = da_spmm_select(&f);
        if (id < 0) throw DaError(-id);
        algo.emplace_back(N, id);
        return id;
    }

    void prepare() { prepare(*now()); }
    void prepare(const Arrays& a) {
        std::lock_guard<std::recursive_mutex> lk(mu);
        if (prepared) return;
        check(da_spmm_prepare(a.m, a.k, a.nnz, data<int32_t>(a.rowptr), data<int32_t>(a.colind), stream_of(a.rowptr)));
        prepared = true;
    }

    std::shared_ptr<Graph> transposed() {
        std::lock_guard<std::recursive_mutex> lk(mu);
        if (auto back = t_of.lock()) return back;
        if (!t) {
            const ArraysPtr a = now();
            c10::DeviceGuard guard(a->rowptr.device());
            Tensor trp = at::empty({a->k + 1}, a->rowptr.options()), tci = at::empty({a->nnz}, a->colind.options()),
                   tva = at::empty({a->nnz}, a->vals.options());
            size_t bytes = 0;
            check(da_csr_transpose_workspace(a->m, a->k, a->nnz, &bytes));
            // scratch of the call; torch allocations are 512-byte aligned and the caching allocator keeps the
            // block alive for work already queued on this stream
            Tensor ws = at::empty({(int64_t)bytes}, a->rowptr.options().dtype(at::kByte));
            check(da_csr_transpose(a->m, a->k, a->nnz, data<int32_t>(a->rowptr), data<int32_t>(a->colind), data<float>(a->vals),
                                   data<int32_t>(trp), data<int32_t>(tci), data<float>(tva), data<void>(ws), bytes,
                                   stream_of(a->rowptr)));
            t = std::make_shared<Graph>(a->k, a->m, trp, tci, tva);
            t->t_of = weak_from_this();
        }
        return t;
    }

    // a . X for X with unit column stride, a = this graph's arrays.  The matrix is prepared (chunk order of the EB
    // algorithms) before the second product with an EB algorithm that the selector chose, and before the first one
    // the caller chose, unless the stream is being captured: preparing allocates and waits, and its orders only
    // cost speed where they are missing.  bias, relu: what a layer does to the sums.
    Tensor product(const Arrays& a, const Tensor& X, int64_t N, std::optional<int> given = std::nullopt,
                   const Tensor& bias = Tensor(), bool relu = false) {
        c10::DeviceGuard guard(a.rowptr.device());
        const int id = given ? *given : algo_for(N);
        if (id >= DA_EB_RM_SR && !prepared && !capturing(a.rowptr)) {
            std::lock_guard<std::recursive_mutex> lk(mu);
            if (given || eb_products > 0) prepare(a);
            ++eb_products;
        }
        Tensor C = at::empty({a.m, N}, a.vals.options());
        check(da_spmm_layer(a.m, a.k, N, data<int32_t>(a.rowptr), data<int32_t>(a.colind), data<float>(a.vals), data<float>(X),
                            leading(X), data<float>(C), data<float>(bias), relu ? 1 : 0, id, stream_of(a.rowptr)));
        return C;
    }
};
using GraphPtr = std::shared_ptr<Graph>;

GraphPtr make_graph(int64_t m, int64_t k, const Tensor& rowptr, const Tensor& colind, const Tensor& vals, bool restored) {
    if (restored) return std::make_shared<Graph>(m, k, rowptr, colind, vals);   // from a copy or file, wherever that left them
    if (rowptr.scalar_type() != at::kInt || colind.scalar_type() != at::kInt || vals.scalar_type() != at::kFloat)
        throw py::type_error("rowptr / colind must be int32 and vals float32");
    if (!(rowptr.is_cuda() && colind.is_cuda() && vals.is_cuda())) throw py::value_error("CSR arrays must live on the GPU");
    if (rowptr.numel() != m + 1 || colind.numel() != vals.numel()) throw py::value_error("CSR array sizes do not match");
    return std::make_shared<Graph>(m, k, rowptr, colind, vals);
}

// X as the product takes it: float32, k rows, neighbouring columns
Tensor operand(const Arrays& a, const Tensor& X) {
    if (X.scalar_type() != at::kFloat || X.dim() != 2 || X.size(0) != a.k) throw py::value_error("X must be a float32 k x N tensor");
    if (X.device() != a.rowptr.device()) throw py::value_error("X must be on the device of the graph");
    return X.resolve_neg().contiguous();
}

// Whether torch does nothing around an operation but differentiate backwards: no tracer that records, no mode
// and no function transform that intercepts
bool ordinary_context() {
    return !torch::jit::tracer::isTracing() && !c10::impl::TorchDispatchModeTLS::any_modes_set() &&
           !at::impl::torch_function_mode_enabled() &&
           !c10::impl::tls_is_dispatch_key_included(c10::DispatchKey::FuncTorchDynamicLayerFrontMode);
}

// Whether a tensor is its memory and nothing else: no wrapper, no lazy negation, no tangent
bool ordinary(const Tensor& t) {
    constexpr c10::DispatchKeySet wrapped(
        {c10::DispatchKey::Python, c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::FuncTorchGradWrapper,
         c10::DispatchKey::Functionalize, c10::DispatchKey::Negative, c10::DispatchKey::Conjugate, c10::DispatchKey::ZeroTensor});
    return t.layout() == at::kStrided && !t.key_set().has_any(wrapped) && !t._fw_grad(0).defined();
}

// ... and its Python object is a Tensor or Parameter, no subclass that overrides operations
bool ordinary(py::handle x) { return THPVariable_CheckExact(x.ptr()) && ordinary(THPVariable_Unpack(x.ptr())); }

struct AggregateBackward : torch::autograd::Node {
    GraphPtr graph;
    torch::autograd::variable_list apply(torch::autograd::variable_list&& grads) override {
        return in_backward([&] { return gradients(grads); });
    }
    torch::autograd::variable_list gradients(const torch::autograd::variable_list& grads) {
        if (!grads[0].defined() || !task_should_compute_output(0)) return {Tensor()};
        at::AutoDispatchBelowADInplaceOrView below;
        const auto t = graph->transposed();
        const ArraysPtr at_now = t->now();
        const Tensor dY = operand(*at_now, grads[0].detach());
        return {t->product(*at_now, dY, dY.size(1))};
    }
    std::string name() const override { return "AggregateBackward"; }
};

bool wants_grad(const Tensor& t) { return t.defined() && t.requires_grad(); }

// x: X as operand() gives it
Tensor aggregate(const GraphPtr& g, const Arrays& a, const Tensor& X, const Tensor& x) {
    Tensor Y;
    {
        at::AutoDispatchBelowADInplaceOrView below;
        Y = g->product(a, x, x.size(1));
    }
    if (at::GradMode::is_enabled() && wants_grad(X)) {
        auto node = std::shared_ptr<AggregateBackward>(new AggregateBackward(), torch::autograd::deleteNode);
        node->graph = g;
        node->set_next_edges(torch::autograd::collect_next_edges(X));
        torch::autograd::set_history(Y, node);
    }
    return Y;
}

// Whether bf16 pieces are the best way for rows x k times k x n.
// Up to 192 inner positions: from some 5000 weights on where the fp32 matrix cores are the bound (100 000 rows: 128 x 128 55 us on
// them, 36 in pieces; 262 144 rows: 128 x 41 49 and 42, 64 x 32 22 and 24), if that pays for the launch that lays the weights
// out (100 003 rows: 96 x 64 25 and 23, but a training step of such a layer 294 and 299); below 64 positions C is most of the
// traffic, which the fp32 kernel writes faster (200 000 rows, 32 x 256: 56 and 64; 300 000, 32 x 512: 255 and 170).
// Up to 256 the fp32 kernel has its weights in LDS for few columns and saves a launch (256 x 16: 1000 rows 7.1 and 11.0,
// 100 000 22.7 and 27.5, 300 000 67.7 and 60.7; 256 x 41: 10 000 rows 11.6 and 13.0, 30 000 17.2 and 14.2; 256 x 64: 12.8 and 12.2).
// Beyond, the library: a block of pieces has 128 rows and walks the whole sum, so few rows of long sums are the library's,
// which splits them (layers, with the library's host time: 602 x 128: 5000 rows 25 and 28; 400 x 128: 15 000 27 and 30; 1000 x 8:
// 40 000 35 and 41; kernels alone: 602 x 128: 20 000 rows 44 and 40, 262 144 358 and 259; 602 x 24: 100 000 116 and 54).
bool pieces_pay(int64_t rows, int64_t k, int64_t n) {
    if (k < 32 || n > 512) return false;
    if (k <= 192) return k * n >= 5000 && rows * k * n >= (k < 64 ? 1800000000 : 1000000000);
    if (k <= 256) return n > (rows < 20000 ? 48 : rows < 200000 ? 16 : rows < 250000 || k < 224 ? 8 : 0);
    return rows >= (n <= 16 && k >= 900 ? 50 : n == 96 || n == 128 ? 40 : 30) * k;
}

// A . W, into `out` (unit column stride): bf16 pieces, the fp32 kernel, which keeps the weights in LDS (up to 128 inner positions,
// and up to 256 for few columns and where the library's 18 us of host time are the larger part), or the GEMM library.
void dense_product(const Tensor& A, const Tensor& W, bool transpose_w, Tensor& out) {
    const int64_t rows = A.size(0), k = A.size(1), n = out.size(1);
    if (A.stride(1) == 1 && W.is_contiguous()) {
        const int64_t wk = transpose_w ? 1 : n, wn = transpose_w ? k : 1;
        size_t bytes = 0;
        if (pieces_pay(rows, k, n) && da_spmm_dense_split_workspace(k, n, &bytes) == DA_OK) {
            Tensor ws = at::empty({(int64_t)bytes}, A.options().dtype(at::kByte));
            const int st = da_spmm_dense_split(rows, k, n, data<float>(A), leading(A), data<float>(W), wk, wn, data<float>(out),
                                               leading(out), data<void>(ws), bytes, stream_of(A));
            if (st != DA_ERR_UNSUPPORTED) return check(st);
        } else if (k >= 1 && (k <= 128 || (k <= 256 && (n <= 16 || rows * k * n <= 300000000)))) {
            const int st = da_spmm_dense(rows, k, n, data<float>(A), leading(A), data<float>(W), wk, wn, data<float>(out),
                                         leading(out), stream_of(A));
            if (st != DA_ERR_UNSUPPORTED) return check(st);
        }
    }
    at::mm_out(out, A, transpose_w ? W.t() : W);
}

// dW = X^T . G.  The own kernel splits the rows over the blocks and wins while there are few tiles of 64 x 64 to dW
// (100 003 rows: 96 x 64 29 us, the library 301; 512 x 256, 32 tiles, 322 and 888).  From 64 tiles on the library's
// tiles reuse more (512 x 512: 627 and 568; 1024 x 1024: 2550 and 1780; 2000 rows of 1024 x 1024: 80 and 40).
// Sizes that the kernels' grids or counters do not hold are refused and the library's too.
Tensor weight_gradient(const Tensor& X, const Tensor& G) {
    const int64_t rows = X.size(0), fin = X.size(1), fout = G.size(1);
    size_t bytes = 0;
    const bool few = ((fin + 63) / 64) * ((fout + 63) / 64) < 64;
    if (rows >= 1 && fin >= 4 && fout >= 4 && few && X.stride(1) == 1 && G.stride(1) == 1) {
        const int st = da_spmm_weight_grad_workspace(rows, fin, fout, &bytes);
        if (st != DA_ERR_UNSUPPORTED) {
            check(st);
            Tensor dW = at::empty({fin, fout}, X.options());
            Tensor ws = at::empty({(int64_t)bytes}, X.options().dtype(at::kByte));
            check(da_spmm_weight_grad(rows, fin, fout, data<float>(X), leading(X), data<float>(G), leading(G), data<float>(dW),
                                      data<void>(ws), bytes, stream_of(X)));
            return dW;
        }
    }
    return at::mm(X.t(), G);
}

// Column sums; sizes that the kernel does not hold are the library's.
Tensor column_sums(const Tensor& G) {
    size_t bytes = 0;
    const int st = da_spmm_column_sums_workspace(G.size(0), G.size(1), &bytes);
    if (st == DA_ERR_UNSUPPORTED) return G.sum(0);
    check(st);
    Tensor sums = at::empty({G.size(1)}, G.options());
    Tensor ws = at::empty({(int64_t)bytes}, G.options().dtype(at::kByte));
    check(da_spmm_column_sums(G.size(0), G.size(1), data<float>(G), leading(G), data<float>(sums), data<void>(ws), bytes,
                              stream_of(G)));
    return sums;
}

// Z = A . (X . W) + b, out = relu(Z):  dZ = dY where out > 0;  db = column sums of dZ;  dH = A^T . dZ;
// dW = X^T . dH;  dX = dH . W^T.  X is kept for dW only and W for dX only: the caller may change or drop what no
// gradient needs.
struct GraphConvBackward : torch::autograd::Node {
    GraphPtr graph;
    torch::autograd::SavedVariable x, w, out;
    bool relu = false;

    void release_variables() override {
        std::lock_guard<std::mutex> lk(mutex_);
        x.reset_data();
        w.reset_data();
        out.reset_data();
    }

    torch::autograd::variable_list apply(torch::autograd::variable_list&& grads) override {
        return in_backward([&] { return gradients(grads); });
    }
    torch::autograd::variable_list gradients(const torch::autograd::variable_list& grads) {
        torch::autograd::variable_list result(3);
        if (!grads[0].defined()) return result;
        const Tensor dY = grads[0].resolve_neg();
        Tensor X, W, Y;
        {
            std::lock_guard<std::mutex> lk(mutex_);
            if (task_should_compute_output(1)) X = x.unpack();
            if (task_should_compute_output(0)) W = w.unpack();
            if (relu) Y = out.unpack(shared_from_this());
        }
        c10::DeviceGuard guard(graph->now()->rowptr.device());
        const bool again = at::GradMode::is_enabled();       // gradients of gradients: dense parts differentiable
        Tensor dZ = relu ? at::threshold_backward(dY, Y, 0) : dY;
        if (!again) dZ = dZ.contiguous();                    // once for all that read it
        if (task_should_compute_output(2)) {
            if (again) result[2] = dZ.sum(0);
            else { at::AutoDispatchBelowADInplaceOrView below; result[2] = column_sums(dZ); }
        }
        if (!task_should_compute_output(0) && !task_should_compute_output(1)) return result;
        Tensor dH;
        {
            at::AutoDispatchBelowADInplaceOrView below;
            const auto t = graph->transposed();
            const ArraysPtr at_now = t->now();
            dH = t->product(*at_now, operand(*at_now, dZ.detach()), dZ.size(1));
        }
        if (again) {
            if (task_should_compute_output(1)) result[1] = at::mm(X.t(), dH);
            if (task_should_compute_output(0)) result[0] = at::mm(dH, W.t());
            return result;
        }
        at::AutoDispatchBelowADInplaceOrView below;
        if (task_should_compute_output(1)) result[1] = weight_gradient(X, dH);
        if (task_should_compute_output(0)) {
            result[0] = at::empty({dH.size(0), W.size(0)}, dH.options());
            dense_product(dH, W, true, result[0]);
        }
        return result;
    }
    std::string name() const override { return "GraphConvBackward"; }
};

Tensor graph_conv(const GraphPtr& g, const Tensor& X, const Tensor& W, const std::optional<Tensor>& bias, bool relu) {
    const Tensor b = bias.value_or(Tensor());
    Tensor Z;
    const int64_t n = W.size(1);
    const ArraysPtr a = g->now();
    if (X.size(0) != a->k) throw py::value_error("X must be a float32 k x N tensor");
    {
        at::AutoDispatchBelowADInplaceOrView below;
        c10::DeviceGuard guard(a->rowptr.device());
        Tensor H = at::empty({X.size(0), row_pitch(n)}, X.options()).narrow(1, 0, n);
        dense_product(X, W, false, H);
        Z = g->product(*a, H, n, std::nullopt, b, relu);
    }
    if (at::GradMode::is_enabled() && (wants_grad(X) || wants_grad(W) || wants_grad(b))) {
        auto node = std::shared_ptr<GraphConvBackward>(new GraphConvBackward(), torch::autograd::deleteNode);
        node->graph = g;
        node->relu = relu;
        if (wants_grad(W)) node->x = torch::autograd::SavedVariable(X, false);
        if (wants_grad(X)) node->w = torch::autograd::SavedVariable(W, false);
        node->set_next_edges(torch::autograd::collect_next_edges(X, W, b));
        torch::autograd::set_history(Z, node);
        if (relu) node->out = torch::autograd::SavedVariable(Z, true);
    }
    return Z;
}

// Whether graph_conv takes these operands as they are (anything else goes the way of separate operations)
bool graph_conv_takes(const GraphPtr& g, py::handle x, py::handle w, py::handle bias) {
    if (!ordinary_context() || at::autocast::is_autocast_enabled(at::kCUDA)) return false;
    if (!ordinary(x) || !ordinary(w) || !(bias.is_none() || ordinary(bias))) return false;
    const ArraysPtr a = g->now();
    auto plain = [&](const Tensor& t, int64_t dim) {
        return t.scalar_type() == at::kFloat && t.dim() == dim && t.is_contiguous() && t.device() == a->rowptr.device();
    };
    const Tensor &X = THPVariable_Unpack(x.ptr()), &W = THPVariable_Unpack(w.ptr());
    return plain(X, 2) && plain(W, 2) && X.size(0) == a->k && X.size(1) == W.size(0) && W.size(1) >= 1 && X.size(1) >= 1 &&
           a->m >= 1 && (bias.is_none() || (plain(THPVariable_Unpack(bias.ptr()), 1) &&
                                            THPVariable_Unpack(bias.ptr()).size(0) == W.size(1)));
}

void bind_graphs(py::module_& mod) {
    py::register_exception_translator([](std::exception_ptr p) {
        try {
            if (p) std::rethrow_exception(p);
        } catch (const DaError& e) {
            set_error(e);
        }
    });
    using release = py::call_guard<py::gil_scoped_release>;
    auto get = [](auto field) { return [field](Graph& g) { return (*g.now()).*field; }; };
    auto put = [](auto field) { return [field](Graph& g, decltype(Arrays{}.*field) value) { g.change(field, value); }; };
    py::class_<Graph, GraphPtr>(mod, "Graph")
        .def(py::init(&make_graph), py::arg("m"), py::arg("k"), py::arg("rowptr"), py::arg("colind"), py::arg("vals"),
             py::arg("restored") = false)
        .def_property("m", get(&Arrays::m), put(&Arrays::m))
        .def_property("k", get(&Arrays::k), put(&Arrays::k))
        .def_property("nnz", get(&Arrays::nnz), put(&Arrays::nnz))
        .def_property("rowptr", get(&Arrays::rowptr), put(&Arrays::rowptr))
        .def_property("colind", get(&Arrays::colind), put(&Arrays::colind))
        .def_property("vals", get(&Arrays::vals), put(&Arrays::vals))
        .def_property_readonly("prepared", [](Graph& g) { return g.prepared.load(); })
        .def("features", [](Graph& g) {
            da_features f;
            { py::gil_scoped_release r; f = g.known(); }
            return py::make_tuple(f.rows, f.nnz, f.row_nnz_mean, f.row_nnz_std, f.row_nnz_max);
        })
        .def("algo_for", &Graph::algo_for, release())
        .def("prepare", [](Graph& g) { g.prepare(); }, release())
        .def("transposed", &Graph::transposed, release())
        .def("spmm", [](Graph& g, const Tensor& X, std::optional<int> id) {
            const ArraysPtr a = g.now();
            const Tensor x = operand(*a, X);
            py::gil_scoped_release r;
            at::AutoDispatchBelowADInplaceOrView below;
            return g.product(*a, x, x.size(1), id);
        });
    mod.def("aggregate", [](const GraphPtr& g, const Tensor& X) {
        const ArraysPtr a = g->now();
        const Tensor x = operand(*a, X);      // errors are Python exceptions: raised with the lock held
        py::gil_scoped_release r;
        return aggregate(g, *a, X, x);
    });
    mod.def("aggregate_takes", [](py::handle X) { return ordinary_context() && ordinary(X); });
    mod.def("graph_conv", &graph_conv, release());
    mod.def("graph_conv_takes", &graph_conv_takes);
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

PyMODINIT_FUNC PyInit__native(void) {
    PyObject* m = PyModule_Create(&kModule);
    if (!m) return nullptr;
    try {
        auto mod = py::reinterpret_borrow<py::module_>(m);
        bind_graphs(mod);
    } catch (const std::exception& e) {
        Py_DECREF(m);
        PyErr_SetString(PyExc_ImportError, e.what());
        return nullptr;
    }
    return m;
}
