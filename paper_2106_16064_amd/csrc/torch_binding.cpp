// Calls from PyTorch into libdgsp without an interpreter step per argument.
//
// A product of a small matrix is bound by the host: 4096 rows of 8 at N = 4 take the GPU 5.6 us, while checking five
// tensors, looking up the stream and converting eleven arguments in Python took 12 us.  Here the same checks read the
// tensors' fields, and a differentiable product is a graph node of its own (forward and backward of a 65 536-vertex graph
// at N = 41: 66 us on the GPU, 137 us of host time through a Python autograd function).
//
// Argument marshalling only: every step of the multiplication runs in libdgsp.  The functions take positional arguments
// (the Python side, binding.py and autograd.py, documents them) and raise the DgspError handed to set_error_type().
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/hip/EmptyTensor.h>
#include <c10/core/DeviceGuard.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPCachingAllocator.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/Stream.h>
#include <torch/csrc/autograd/function.h>
#include <torch/csrc/autograd/functions/utils.h>
#include <torch/csrc/autograd/grad_mode.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/jit/frontend/tracer.h>

#include <cstring>
#include <optional>
#include <string>

#include "dgsp_internal.h"
#include "workspace.hpp"

namespace {

PyObject* g_error = nullptr;      // DgspError, a strong reference for the life of the process

// A Python exception is set: unwinds to the function's entry.
struct Raised {};

[[noreturn]] void fail(const std::string& what) {
    PyErr_SetString(g_error ? g_error : PyExc_RuntimeError, what.c_str());
    throw Raised{};
}

void check_status(int rc, const char* what) {
    if (rc != DGSP_OK) fail(std::string(what) + ": " + dgsp_status_string(rc) + " (status " + std::to_string(rc) + ")");
}

int64_t as_int(PyObject* o) {
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw Raised{};
    return v;
}

// Entry counts, algos and factors: what int() and float() take.
int64_t to_int(PyObject* o) {
    if (PyLong_CheckExact(o)) return as_int(o);
    PyObject* i = PyNumber_Long(o);
    if (!i) throw Raised{};
    const long long v = PyLong_AsLongLong(i);
    Py_DECREF(i);
    if (v == -1 && PyErr_Occurred()) throw Raised{};
    return v;
}

float to_float(PyObject* o) {
    if (PyFloat_CheckExact(o)) return (float)PyFloat_AS_DOUBLE(o);
    PyObject* f = PyNumber_Float(o);
    if (!f) throw Raised{};
    const double v = PyFloat_AS_DOUBLE(f);
    Py_DECREF(f);
    return (float)v;
}

const at::Tensor& as_tensor(PyObject* o, const char* name) {
    if (!THPVariable_Check(o)) {
        fail(std::string(name) + " must be a tensor");
    }
    return THPVariable_Unpack(o);
}

// The stream that a call runs on; `known`: as torch's allocator knows it, none for a stream that is not torch's, which may be gone
// when the allocator asks how far it has come.
struct CallStream {
    void* handle;
    std::optional<c10::hip::HIPStream> known;
};

CallStream call_stream(c10::hip::HIPStream s) {
    void* handle = s.stream();
    const bool foreign = handle != nullptr && s.id() == (int64_t)reinterpret_cast<intptr_t>(handle);      // named by their address
    return {handle, foreign ? std::nullopt : std::make_optional(s)};
}

CallStream current_stream() { return call_stream(c10::hip::getCurrentHIPStream()); }

// the torch stream given, or the current one
CallStream as_stream(PyObject* o) {
    if (o == Py_None) return current_stream();
    PyObject* handle = PyObject_GetAttrString(o, "cuda_stream");
    if (!handle) throw Raised{};
    void* p = PyLong_AsVoidPtr(handle);
    Py_DECREF(handle);
    if (!p && PyErr_Occurred()) throw Raised{};
    if (!THPStream_Check(o)) return {p, std::nullopt};
    const auto* t = reinterpret_cast<THPStream*>(o);
    const c10::Device device(c10::DeviceType::HIP, (c10::DeviceIndex)t->device_index);
    const c10::Stream named(c10::Stream::UNSAFE, device, t->stream_id);
    const CallStream s = call_stream(c10::hip::HIPStream(c10::hip::HIPStream::UNCHECKED, named));
    return s.handle == p ? s : CallStream{p, std::nullopt};
}

void* ptr(const at::Tensor& t) { return t.numel() == 0 ? nullptr : t.data_ptr(); }

// the matrix arrays of the entry points that leave their checks to the library: None is a null pointer
void* ptr(PyObject* o, const char* name) { return o == Py_None ? nullptr : ptr(as_tensor(o, name)); }

bool on_gpu(const at::Tensor& t) { return t.device().is_cuda() && t.layout() == at::kStrided; }

bool is_array(const at::Tensor& t, at::ScalarType type) { return on_gpu(t) && t.scalar_type() == type && t.is_contiguous(); }

// what Workspace asks
struct HipRuntime {
    using Stream = hipStream_t;
    static bool capture_status(Stream stream, bool& recording) {
        hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
        const bool known = hipStreamIsCapturing(stream, &status) == hipSuccess;
        recording = status != hipStreamCaptureStatusNone;
        return known;
    }
    static bool device(int& d) { return hipGetDevice(&d) == hipSuccess; }
    static bool device_of(Stream stream, int& d) {
        hipDevice_t on = -1;
        const bool known = hipStreamGetDevice(stream, &on) == hipSuccess;
        d = on;
        return known;
    }
    static void* allocate(size_t bytes, Stream stream) { return c10::hip::HIPCachingAllocator::raw_alloc_with_stream(bytes, stream); }
    static void release(void* memory) { c10::hip::HIPCachingAllocator::raw_delete(memory); }
    static void forget_error() { (void)hipGetLastError(); }
};
using Workspace = dgsp::Workspace<HipRuntime>;

// would any product look at the table?
bool wants_hot_columns(const dgsp_internal_stats_t& stats) {
    for (int64_t n = 1; n <= 4; ++n)
        if (stats.hot_share[n - 1] > 0.0 && dgsp_internal_wants_hot_columns(&stats, n)) return true;
    return false;
}

// The statistics of a ctypes `Features` structure, or of the `MatrixFeatures` that a DeviceCsr holds (None: there are none).
class FeaturesArg {
public:
    explicit FeaturesArg(PyObject* o) {
        if (o == Py_None) return;
        Py_buffer view;
        if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) throw Raised{};
        const bool fits = view.len == (Py_ssize_t)sizeof(value_) || view.len == (Py_ssize_t)sizeof(value_.features);
        if (fits) memcpy(&value_, view.buf, (size_t)view.len);
        PyBuffer_Release(&view);
        if (!fits) {
            PyErr_SetString(PyExc_TypeError, "features must be a Features structure");
            throw Raised{};
        }
        given_ = true;
        if (wants_hot_columns(value_)) take_hot_columns(o);
    }
    const dgsp_features_t* get() const { return given_ ? &value_.features : nullptr; }
    // for a product with N columns on the GPU of `X`
    dgsp_internal_hints_t hints(int64_t N, const at::Tensor& X, Workspace& workspace, const CallStream& stream) const {
        return {value_.saved_share, hot_columns(N, X, stream), &Workspace::get, &workspace};
    }

private:
    // The table goes when the structure does, which the caller may let go as soon as the call has returned.  Its memory must not be
    // handed out again before the product has run: on the stream that it was allocated on it comes later anyway, other streams of
    // torch's are named to the allocator, and on those that torch does not know products go the general way.  So do products that are
    // recorded into a graph: its replays read whatever has become of the table.
    const uint32_t* hot_columns(int64_t N, const at::Tensor& X, const CallStream& stream) const {
        if (!hot_.defined() || hot_.device() != X.device() || !dgsp_internal_wants_hot_columns(&value_, N)) return nullptr;
        bool recording = false;
        if (!HipRuntime::capture_status(static_cast<hipStream_t>(stream.handle), recording)) {
            HipRuntime::forget_error();
            return nullptr;
        }
        if (recording) return nullptr;
        if (!stream.handle || stream.handle != hot_stream_) {
            if (!stream.known) return nullptr;
            c10::hip::HIPCachingAllocator::recordStream(hot_.storage().data_ptr(), *stream.known);
        }
        return static_cast<const uint32_t*>(hot_.data_ptr());
    }

    // A tensor that the structure carries as an attribute and not as an address among its bytes, which could outlive it.
    void take_hot_columns(PyObject* o) {
        static PyObject* const columns = PyUnicode_InternFromString("hot_columns");
        static PyObject* const stream = PyUnicode_InternFromString("hot_stream");
        PyObject *t = PyObject_GetAttr(o, columns), *s = t ? PyObject_GetAttr(o, stream) : nullptr;
        if (t && THPVariable_Check(t)) {
            const at::Tensor& table = THPVariable_Unpack(t);
            if (is_array(table, at::kInt) && table.numel() * 4 == dgsp_internal_hot_columns_bytes(&value_)) hot_ = table;
        }
        if (s && PyLong_Check(s)) hot_stream_ = PyLong_AsVoidPtr(s);
        PyErr_Clear();
        Py_XDECREF(s);
        Py_XDECREF(t);
    }

    dgsp_internal_stats_t value_{};
    bool given_ = false;
    at::Tensor hot_;
    void* hot_stream_ = nullptr;
};

void check_array(const at::Tensor& t, at::ScalarType type, const char* name, const char* type_name) {
    if (!is_array(t, type)) fail(std::string(name) + " must be a contiguous " + type_name + " tensor on the GPU");
}

void check_csr(int64_t M, const at::Tensor& rowptr, const at::Tensor& colidx, const at::Tensor& vals) {
    check_array(rowptr, at::kInt, "rowptr", "torch.int32");
    check_array(colidx, at::kInt, "colidx", "torch.int32");
    check_array(vals, at::kFloat, "vals", "torch.float32");
    if (rowptr.numel() != M + 1 || colidx.numel() != vals.numel())
        fail("rowptr needs M+1 entries; colidx and vals must have equal length");
}

void check_packed(int64_t M, int64_t K, int64_t N, const at::Tensor& X, const at::Tensor& Y) {
    check_array(X, at::kFloat, "X", "torch.float32");
    check_array(Y, at::kFloat, "Y", "torch.float32");
    if (X.numel() != K * N || Y.numel() != M * N) fail("X must hold K*N and Y M*N elements");
}

// leading dimension of a 2-D view with unit column stride
int64_t check_view(const at::Tensor& t, const char* name, int64_t rows, int64_t cols) {
    if (!on_gpu(t) || t.scalar_type() != at::kFloat || t.dim() != 2 || (t.size(1) > 1 && t.stride(1) != 1))
        fail(std::string(name) + " must be a 2-D float32 GPU view with unit column stride");
    if (t.size(0) != rows || t.size(1) != cols) fail("X must be K x N and Y M x N");
    return rows > 1 ? t.stride(0) : std::max(cols, t.stride(0));
}

// The library call itself, with the interpreter lock released: a full queue can make a launch wait.
template <typename F>
int unlocked(F&& call) {
    PyThreadState* state = PyEval_SaveThread();
    const int rc = call();
    PyEval_RestoreThread(state);
    return rc;
}

// what is known of a matrix when it has been taken over
struct Measured {
    dgsp_internal_stats_t stats{};
    at::Tensor hot_columns;         // undefined: none, or none worth having
    void* hot_stream = nullptr;     // that its memory belongs to
};

void write_features(PyObject* o, const Measured& m) {
    const dgsp_internal_stats_t& f = m.stats;
    Py_buffer view;
    if (PyObject_GetBuffer(o, &view, PyBUF_WRITABLE) != 0) throw Raised{};
    const bool fits = view.len == (Py_ssize_t)sizeof(f);
    if (fits) memcpy(view.buf, &f, sizeof(f));
    PyBuffer_Release(&view);
    if (!fits) fail("features must be a MatrixFeatures structure");
    if (m.hot_columns.defined()) {
        PyObject* table = THPVariable_Wrap(m.hot_columns);
        PyObject* stream = PyLong_FromVoidPtr(m.hot_stream);
        const bool set = table && stream && PyObject_SetAttrString(o, "hot_columns", table) == 0 &&
                         PyObject_SetAttrString(o, "hot_stream", stream) == 0;
        Py_XDECREF(stream);
        Py_XDECREF(table);
        if (!set) throw Raised{};
    }
}

// ---------------------------------------------------------------- one product

// Y = A X by a named kernel, or by the rules (DGSP_AUTO); returns the status and leaves the kernel run in `algo`
int product(int64_t M, int64_t K, int64_t N, const FeaturesArg& f, const at::Tensor& rowptr, const at::Tensor& colidx,
            const at::Tensor& vals, const at::Tensor& X, const at::Tensor& Y, int& algo, const CallStream& on) {
    const auto* rp = static_cast<const int32_t*>(ptr(rowptr));
    const auto* ci = static_cast<const int32_t*>(ptr(colidx));
    const auto* av = static_cast<const float*>(ptr(vals));
    const auto* x = static_cast<const float*>(ptr(X));
    auto* y = static_cast<float*>(ptr(Y));
    void* const stream = on.handle;
    Workspace workspace(static_cast<hipStream_t>(stream), X.device().index());
    const dgsp_internal_hints_t hints = f.hints(N, X, workspace, on);
    if (algo == DGSP_AUTO) return dgsp_internal_spmm_auto(M, K, N, f.get(), &hints, rp, ci, av, x, y, &algo, stream);
    return dgsp_internal_spmm_phase(M, K, N, colidx.numel(), rp, ci, av, x, y, algo, DGSP_PHASE_ALL, f.get(), &hints, stream);
}

// M x N, or M elements when the dense operand is a vector.  A GPU tensor comes from the allocator directly: the dispatcher's
// way there is 0.3 us of a 4.5 us call.
at::Tensor empty_result(int64_t M, int64_t N, bool vector, const at::Tensor& like) {
    const int64_t sizes[2] = {M, N};
    const at::IntArrayRef shape(sizes, vector ? 1 : 2);
    if (!like.device().is_cuda()) return at::empty(shape, at::TensorOptions().dtype(at::kFloat).device(like.device()));
    return at::Tensor(at::detail::empty_cuda(shape, at::kFloat, like.device(), std::nullopt));
}

int64_t columns_of(const at::Tensor& X) { return X.dim() == 2 ? X.size(1) : 1; }

struct Csr {
    int64_t M, K;
    FeaturesArg features;
    at::Tensor rowptr, colidx, vals;
    // a[0 ... 3]: features, rowptr, colidx, vals
    Csr(PyObject* const* a, int64_t rows, int64_t cols)
        : M(rows), K(cols), features(a[0]), rowptr(as_tensor(a[1], "rowptr")), colidx(as_tensor(a[2], "colidx")),
          vals(as_tensor(a[3], "vals")) {
        if (!features.get()) fail("the matrix has no features");
        check_csr(M, rowptr, colidx, vals);
    }
};

// on the current stream; called with the interpreter lock held
at::Tensor multiply(const Csr& A, const at::Tensor& X, int algo, bool vector_result) {
    const int64_t N = columns_of(X);
    at::Tensor Y = empty_result(A.M, N, vector_result, X);
    check_packed(A.M, A.K, N, X, Y);
    const CallStream stream = current_stream();
    const int rc = unlocked([&] { return product(A.M, A.K, N, A.features, A.rowptr, A.colidx, A.vals, X, Y, algo, stream); });
    check_status(rc, "dgsp_spmm_csr_auto");
    return Y;
}

// dX = A^T dY in autograd's graph.  Not differentiable itself, as the product's kernels are not.
struct ProductBackward : public torch::autograd::Node {
    Csr transposed;
    int algo;
    bool vector;
    ProductBackward(Csr t, int algo_, bool vector_) : transposed(std::move(t)), algo(algo_), vector(vector_) {}

    torch::autograd::variable_list apply(torch::autograd::variable_list&& grads) override {
        if (!grads[0].defined()) return {at::Tensor()};
        at::NoGradGuard no_grad;
        const Csr& A = transposed;
        const at::Tensor G = grads[0].to(at::kFloat).contiguous();
        const int64_t N = vector ? 1 : G.size(1);
        TORCH_CHECK(on_gpu(G) && G.numel() == A.K * N, "the gradient must be a GPU tensor of M*N elements");
        const at::Tensor dX = empty_result(A.M, N, vector, G);
        int which = algo;
        const int rc = product(A.M, A.K, N, A.features, A.rowptr, A.colidx, A.vals, G, dX, which,
                               current_stream());
        TORCH_CHECK(rc == DGSP_OK, "dgsp_spmm_csr_auto: ", dgsp_status_string(rc), " (status ", rc, ")");
        return {dX};
    }
    std::string name() const override { return "SpMMBackward"; }
};

// ---------------------------------------------------------------- a matrix from arrays on the GPU

struct CsrArrays { at::Tensor rowptr, colidx, vals; };

// What narrower column blocks save and which runs of columns are the hottest, from the columns on the GPU: a launch and a wait,
// 20 us, where the matrix is one whose products look at it (four million entries and more, very uneven rows).  Here and not in
// the product, which does not wait.
void measure_columns(Measured& m, const at::Tensor& colidx, void* stream) {
    if (colidx.numel() < m.stats.features.nnz) return;
    const auto* columns = static_cast<const int32_t*>(ptr(colidx));
    uint32_t* table = nullptr;
    if (const int64_t bytes = dgsp_internal_hot_columns_bytes(&m.stats)) {
        try {
            m.hot_columns = at::empty({bytes / 4}, colidx.options());
            m.hot_stream = c10::hip::getCurrentHIPStream(colidx.device().index()).stream();
            table = static_cast<uint32_t*>(m.hot_columns.data_ptr());
        } catch (const c10::OutOfMemoryError&) {                                // no table: the general way
            HipRuntime::forget_error();
        }
    }
    const int rc = unlocked([&] { return dgsp_internal_measure_columns(&m.stats, columns, table, stream); });
    if (rc != DGSP_OK) m.stats = dgsp_internal_stats_t{m.stats.features};       // not measured: the general way
    if (!wants_hot_columns(m.stats)) m.hot_columns.reset();
}

// The arrays in the library's types and the statistics, which the call waits for.  int64 indices are narrowed by the
// statistics' own launch.
CsrArrays take_csr(int64_t M, int64_t K, const at::Tensor& rowptr, const at::Tensor& colidx, const at::Tensor& vals,
                   Measured& measured) {
    at::NoGradGuard no_grad;
    dgsp_internal_stats_t& stats = measured.stats;
    CsrArrays out;
    const bool wide = is_array(rowptr, at::kLong) && is_array(colidx, at::kLong) && M > 0 && colidx.numel() < INT32_MAX - 4096;
    out.rowptr = wide ? at::empty(rowptr.sizes(), rowptr.options().dtype(at::kInt)) : rowptr.to(at::kInt).contiguous();
    out.colidx = wide ? at::empty(colidx.sizes(), colidx.options().dtype(at::kInt)) : colidx.to(at::kInt).contiguous();
    out.vals = is_array(vals, at::kFloat) ? vals : vals.to(at::kFloat).contiguous();
    if (!on_gpu(out.rowptr) || !on_gpu(out.colidx) || out.rowptr.numel() != M + 1) fail("rowptr needs M+1 entries on the GPU");
    if (M == 0) {
        stats.features.K = K;
        return out;
    }
    void* stream = c10::hip::getCurrentHIPStream().stream();
    const int64_t entries = colidx.numel();
    const void* rp = ptr(wide ? rowptr : out.rowptr);
    const void* ci = ptr(wide ? colidx : out.colidx);
    auto* rp32 = static_cast<int32_t*>(ptr(out.rowptr));
    auto* ci32 = static_cast<int32_t*>(ptr(out.colidx));
    check_status(unlocked([&] { return dgsp_internal_take_csr(M, K, entries, wide ? 8 : 4, rp, ci, rp32, ci32, &stats.features, stream); }),
                 "dgsp_features_from_csr_device");
    measure_columns(measured, out.colidx, stream);
    return out;
}

// ---------------------------------------------------------------- the functions

void want(Py_ssize_t n, Py_ssize_t expected) {
    if (n != expected) {
        PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", expected, n);
        throw Raised{};
    }
}

template <PyObject* (*F)(PyObject* const*, Py_ssize_t)>
PyObject* entry(PyObject*, PyObject* const* a, Py_ssize_t n) {
    try {
        return F(a, n);
    } catch (const Raised&) {
        return nullptr;
    } catch (...) {                                // out of memory, among others: the exception torch itself would raise
        torch::translate_exception_to_python(std::current_exception());
        return nullptr;
    }
}

PyObject* set_error_type(PyObject* const* a, Py_ssize_t n) {
    want(n, 1);
    Py_INCREF(a[0]);
    Py_XDECREF(g_error);
    g_error = a[0];
    Py_RETURN_NONE;
}

// (M, K, features, rowptr, colidx, vals, X, algo) -> Y
PyObject* multiply_new(PyObject* const* a, Py_ssize_t n) {
    want(n, 8);
    Csr A(a + 2, as_int(a[0]), as_int(a[1]));
    const at::Tensor& X = as_tensor(a[6], "X");
    return THPVariable_Wrap(multiply(A, X, (int)to_int(a[7]), false));
}

// Does nothing but reverse mode look at a product of X?  Not so under a tangent on X (forward mode), a function transform
// (vmap, grad, jvp), a trace that is being recorded, or Python code that intercepts operations: a graph node of our own
// would pass by them and return a result without tangent, batch or record.
bool only_reverse_mode(const at::Tensor& X) {
    const auto included = c10::impl::tls_local_dispatch_key_set().included_;
    return !X._fw_grad(/*level=*/0).defined() && !X.unsafeGetTensorImpl()->is_python_dispatch() &&
           !included.has(c10::DispatchKey::FuncTorchDynamicLayerFrontMode) &&
           !included.has(c10::DispatchKey::FuncTorchDynamicLayerBackMode) && !torch::jit::tracer::isTracing() &&
           !c10::impl::TorchDispatchModeTLS::any_modes_set();
}

// (X, algo, bwd_algo, fwd M, K, features, rowptr, colidx, vals, bwd M, K, features, rowptr, colidx, vals) -> Y with a graph node;
// None: the caller takes the way through autograd's own Function
PyObject* multiply_differentiable(PyObject* const* a, Py_ssize_t n) {
    want(n, 15);
    const at::Tensor& X = as_tensor(a[0], "X");
    if (!only_reverse_mode(X)) Py_RETURN_NONE;
    Csr A(a + 5, as_int(a[3]), as_int(a[4]));
    const bool vector = X.dim() == 1;
    at::Tensor Y;
    {
        at::NoGradGuard no_grad;
        Y = multiply(A, X.to(at::kFloat).contiguous(), (int)to_int(a[1]), vector);
    }
    if (at::GradMode::is_enabled() && X.requires_grad()) {
        Csr T(a + 11, as_int(a[9]), as_int(a[10]));
        std::shared_ptr<ProductBackward> node(new ProductBackward(std::move(T), (int)to_int(a[2]), vector), torch::autograd::deleteNode);
        node->set_next_edges(torch::autograd::collect_next_edges(X));
        torch::autograd::set_history(Y, node);
    }
    return THPVariable_Wrap(std::move(Y));
}

PyObject* wrapped(CsrArrays&& a, int64_t M, int64_t K) {
    PyObject* rowptr = THPVariable_Wrap(std::move(a.rowptr));
    PyObject* colidx = THPVariable_Wrap(std::move(a.colidx));
    PyObject* vals = THPVariable_Wrap(std::move(a.vals));
    return Py_BuildValue("LLNNN", (long long)M, (long long)K, rowptr, colidx, vals);
}

// (M, K, rowptr, colidx, vals, features to fill) -> (M, K, rowptr, colidx, vals) in the library's types
PyObject* csr_from_arrays(PyObject* const* a, Py_ssize_t n) {
    want(n, 6);
    const int64_t M = as_int(a[0]), K = as_int(a[1]);
    Measured f;
    CsrArrays arrays = take_csr(M, K, as_tensor(a[2], "rowptr"), as_tensor(a[3], "colidx"), as_tensor(a[4], "vals"), f);
    write_features(a[5], f);
    return wrapped(std::move(arrays), M, K);
}

// (sparse CSR tensor, features to fill) -> the same
PyObject* csr_from_tensor(PyObject* const* a, Py_ssize_t n) {
    want(n, 2);
    const at::Tensor& T = as_tensor(a[0], "matrix");
    if (T.layout() != at::kSparseCsr || T.dim() != 2) fail("the matrix must be a 2-D sparse CSR tensor");
    Measured f;
    CsrArrays arrays = take_csr(T.size(0), T.size(1), T.crow_indices(), T.col_indices(), T.values().detach(), f);
    write_features(a[1], f);
    return wrapped(std::move(arrays), T.size(0), T.size(1));
}

// (features, colidx): the columns of a matrix whose statistics are from the host; waits for the current stream of its device
PyObject* measure_matrix_columns(PyObject* const* a, Py_ssize_t n) {
    want(n, 2);
    FeaturesArg f(a[0]);
    const at::Tensor& colidx = as_tensor(a[1], "colidx");
    if (f.get() && is_array(colidx, at::kInt)) {
        const c10::DeviceGuard guard(colidx.device());
        Measured m;
        m.stats.features = *f.get();
        measure_columns(m, colidx, c10::hip::getCurrentHIPStream().stream());
        write_features(a[0], m);
    }
    Py_RETURN_NONE;
}

// (M, K, N, nnz, rowptr, colidx, vals, X, Y, algo, phase, features, stream); one step of the multiplication
PyObject* spmm_csr_phase(PyObject* const* a, Py_ssize_t n) {
    want(n, 13);
    const int64_t M = as_int(a[0]), K = as_int(a[1]), N = as_int(a[2]), nnz = to_int(a[3]);
    const int algo = (int)to_int(a[9]), phase = (int)to_int(a[10]);
    const at::Tensor &rowptr = as_tensor(a[4], "rowptr"), &colidx = as_tensor(a[5], "colidx"), &vals = as_tensor(a[6], "vals");
    const at::Tensor &X = as_tensor(a[7], "X"), &Y = as_tensor(a[8], "Y");
    check_csr(M, rowptr, colidx, vals);
    check_packed(M, K, N, X, Y);
    FeaturesArg f(a[11]);
    const CallStream on = as_stream(a[12]);
    void* const stream = on.handle;
    const auto* rp = static_cast<const int32_t*>(ptr(rowptr));
    const auto* ci = static_cast<const int32_t*>(ptr(colidx));
    const auto* av = static_cast<const float*>(ptr(vals));
    const auto* x = static_cast<const float*>(ptr(X));
    auto* y = static_cast<float*>(ptr(Y));
    Workspace workspace(static_cast<hipStream_t>(stream), X.device().index());
    const dgsp_internal_hints_t hints = f.hints(N, X, workspace, on);
    check_status(unlocked([&] {
        return dgsp_internal_spmm_phase(M, K, N, nnz, rp, ci, av, x, y, algo, phase, f.get(), &hints, stream);
    }), "dgsp_spmm_csr_phase");
    Py_RETURN_NONE;
}

// (M, K, N, features, rowptr, colidx, vals, X, Y, stream) -> kernel run
PyObject* spmm_csr_auto(PyObject* const* a, Py_ssize_t n) {
    want(n, 10);
    const int64_t M = as_int(a[0]), K = as_int(a[1]), N = as_int(a[2]);
    FeaturesArg f(a[3]);
    const at::Tensor &rowptr = as_tensor(a[4], "rowptr"), &colidx = as_tensor(a[5], "colidx"), &vals = as_tensor(a[6], "vals");
    const at::Tensor &X = as_tensor(a[7], "X"), &Y = as_tensor(a[8], "Y");
    check_csr(M, rowptr, colidx, vals);
    check_packed(M, K, N, X, Y);
    const CallStream stream = as_stream(a[9]);
    int algo = DGSP_AUTO;
    check_status(unlocked([&] { return product(M, K, N, f, rowptr, colidx, vals, X, Y, algo, stream); }), "dgsp_spmm_csr_auto");
    return PyLong_FromLong(algo);
}

// `a`: rowptr, colidx, vals, X, Y, algo, stream; `count` nullptr: the entry count is read on the device
void packed_product(PyObject* const* extents, PyObject* count, PyObject* const* a) {
    const int64_t M = as_int(extents[0]), K = as_int(extents[1]), N = as_int(extents[2]);
    const int64_t nnz = count ? to_int(count) : -1;
    const int algo = (int)to_int(a[5]);
    const at::Tensor &rowptr = as_tensor(a[0], "rowptr"), &colidx = as_tensor(a[1], "colidx"), &vals = as_tensor(a[2], "vals");
    const at::Tensor &X = as_tensor(a[3], "X"), &Y = as_tensor(a[4], "Y");
    check_csr(M, rowptr, colidx, vals);
    check_packed(M, K, N, X, Y);
    if (nnz >= 0 && colidx.numel() < nnz) fail("colidx/vals shorter than nnz");
    void* const stream = as_stream(a[6]).handle;
    Workspace workspace(static_cast<hipStream_t>(stream), X.device().index());
    const dgsp_internal_hints_t hints = {0.0, nullptr, &Workspace::get, &workspace};
    const auto* rp = static_cast<const int32_t*>(ptr(rowptr));
    const auto* ci = static_cast<const int32_t*>(ptr(colidx));
    const auto* av = static_cast<const float*>(ptr(vals));
    const auto* x = static_cast<const float*>(ptr(X));
    auto* y = static_cast<float*>(ptr(Y));
    const int rc = unlocked([&] {
        return dgsp_internal_spmm_csr(M, K, N, count ? nnz : -1, colidx.numel(), rp, ci, av, x, y, algo, &hints, stream);
    });
    check_status(rc, count ? "dgsp_spmm_csr_nnz" : "dgsp_spmm_csr");
}

// (M, K, N, rowptr, colidx, vals, X, Y, algo, stream)
PyObject* spmm_csr(PyObject* const* a, Py_ssize_t n) {
    want(n, 10);
    packed_product(a, nullptr, a + 3);
    Py_RETURN_NONE;
}

// (M, K, N, nnz, rowptr, colidx, vals, X, Y, algo, stream)
PyObject* spmm_csr_nnz(PyObject* const* a, Py_ssize_t n) {
    want(n, 11);
    packed_product(a, a[3], a + 4);
    Py_RETURN_NONE;
}

// `a`: M, K, N, nnz, rowptr, colidx, vals, X, Y; `b`: algo, features, stream; `factors` alpha and beta, nullptr: the plain product
void view_product(PyObject* const* a, const float* factors, PyObject* const* b) {
    const int64_t M = as_int(a[0]), K = as_int(a[1]), N = as_int(a[2]), nnz = to_int(a[3]);
    const at::Tensor &X = as_tensor(a[7], "X"), &Y = as_tensor(a[8], "Y");
    const int64_t ldx = check_view(X, "X", K, N), ldy = check_view(Y, "Y", M, N);
    const int algo = (int)to_int(b[0]);
    FeaturesArg f(b[1]);
    const CallStream on = as_stream(b[2]);
    void* const stream = on.handle;
    const auto* rp = static_cast<const int32_t*>(ptr(a[4], "rowptr"));
    const auto* ci = static_cast<const int32_t*>(ptr(a[5], "colidx"));
    const auto* av = static_cast<const float*>(ptr(a[6], "vals"));
    const auto* x = static_cast<const float*>(ptr(X));
    auto* y = static_cast<float*>(ptr(Y));
    Workspace workspace(static_cast<hipStream_t>(stream), X.device().index());
    const dgsp_internal_hints_t hints = f.hints(N, X, workspace, on);
    const int rc = unlocked([&] {
        return dgsp_internal_spmm_view(M, K, N, nnz, rp, ci, av, x, ldx, y, ldy, factors, algo, f.get(), &hints, stream);
    });
    check_status(rc, factors ? "dgsp_spmm_csr_axpby" : "dgsp_spmm_csr_ld");
}

// (M, K, N, nnz, rowptr, colidx, vals, X, Y, algo, features, stream)
PyObject* spmm_csr_ld(PyObject* const* a, Py_ssize_t n) {
    want(n, 12);
    view_product(a, nullptr, a + 9);
    Py_RETURN_NONE;
}

// (M, K, N, nnz, rowptr, colidx, vals, X, Y, alpha, beta, algo, features, stream)
PyObject* spmm_csr_axpby(PyObject* const* a, Py_ssize_t n) {
    want(n, 14);
    const float factors[2] = {to_float(a[9]), to_float(a[10])};
    view_product(a, factors, a + 11);
    Py_RETURN_NONE;
}

#define DGSP_ENTRY(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(&entry<name>)), METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {
    DGSP_ENTRY(set_error_type), DGSP_ENTRY(multiply_new), DGSP_ENTRY(multiply_differentiable), DGSP_ENTRY(spmm_csr_auto),
    DGSP_ENTRY(spmm_csr), DGSP_ENTRY(spmm_csr_nnz), DGSP_ENTRY(spmm_csr_ld), DGSP_ENTRY(spmm_csr_axpby), DGSP_ENTRY(spmm_csr_phase),
    DGSP_ENTRY(csr_from_arrays), DGSP_ENTRY(csr_from_tensor), DGSP_ENTRY(measure_matrix_columns), {nullptr, nullptr, 0, nullptr},
};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_dgsp_torch", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__dgsp_torch(void) { return PyModule_Create(&g_module); }
