// Python calls of libdfp4 that allocate their results: arguments are unpacked, results and workspaces allocated and the C entry
// point called in one native call.  (paper_2501_01144_amd/dfp4.py; the entry points themselves are include/dfp4.h.)
// What bounds small products is the host: quantize + dfp4_gemm of 32 x 4096 x 4096 keeps the GPU busy for 14 us and took 21 us
// through ctypes structures and torch.empty calls, 13.4 so (a call that allocates its result: 8 to 12 us of host time, 5 to 7 so).
#include <Python.h>
#include <dlfcn.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/dfp4.h"

namespace {

PyObject* g_error = nullptr;          // Dfp4Error

#define DFP4_FUNCTIONS(F)                                                                                                  \
    F(dfp4_quantize) F(mxfp4_quantize) F(dfp4_quantize_block) F(dfp4_quantize_native) F(dfp4_dequantize) F(mxfp4_dequantize)  \
    F(dfp4_gemm) F(mxfp4_gemm) F(dfp4_gemm_batched) F(dfp4_gemm_workspace_bytes) F(dfp4_gemm_prepared_bytes)                \
    F(dfp4_gemm_prepare) F(mxfp4_gemm_prepare) F(dfp4_gemm_prepared_workspace_bytes) F(dfp4_gemm_prepared)                  \
    F(mxfp4_gemm_prepared) F(dfp4_native_packed_bytes) F(dfp4_native_pack) F(mxfp4_native_pack)                             \
    F(dfp4_gemm_native_packed) F(mxfp4_gemm_native_packed) F(dfp4_gemm_native_splitk_bytes) F(dfp4_strerror)
#define DFP4_DECLARE(NAME) decltype(&::NAME) p_##NAME = nullptr;
DFP4_FUNCTIONS(DFP4_DECLARE)
#undef DFP4_DECLARE

struct Failure {};                    // a Python exception is set

[[noreturn]] void fail(PyObject* type, const char* what) {
    PyErr_SetString(type, what);
    throw Failure{};
}

// Other Python threads run while memory is allocated (which may wait for the GPU) and while kernels are enqueued (a full queue waits)
struct Unlocked {
    PyThreadState* state = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(state); }
};

// an entry point of the library
template <class F, class... A>
void enqueue(const char* what, F* entry, A... a) {
    int rc;
    {
        Unlocked u;
        rc = entry(a...);
    }
    if (rc == DFP4_OK) return;
    PyErr_Format(g_error, "%s failed: %s (%d)", what, p_dfp4_strerror(rc), rc);
    throw Failure{};
}

const at::Tensor& tensor(PyObject* o) {
    if (!THPVariable_Check(o)) fail(PyExc_TypeError, "a tensor is expected");
    return THPVariable_Unpack(o);
}
int64_t number(PyObject* o) {
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw Failure{};
    return v;
}
uint8_t* data(const at::Tensor& t) { return t.numel() > 0 ? static_cast<uint8_t*>(t.data_ptr()) : nullptr; }
uint8_t* data(PyObject* o) { return o == Py_None ? nullptr : data(tensor(o)); }
void* stream() { return c10::hip::getCurrentHIPStream().stream(); }

at::Tensor empty(at::IntArrayRef shape, at::ScalarType type, const at::Device& dev) {
    Unlocked u;
    return at::empty(shape, at::TensorOptions().dtype(type).device(dev));
}
at::Tensor bytes(int64_t n, const at::Device& dev) { return empty({n}, at::kByte, dev); }
at::Tensor bytes(int64_t r, int64_t c, const at::Device& dev) { return empty({r, c}, at::kByte, dev); }
at::Tensor result(at::IntArrayRef shape, bool bf16, const at::Device& dev) { return empty(shape, bf16 ? at::kBFloat16 : at::kFloat, dev); }

int dtype(bool bf16) { return bf16 ? DFP4_BF16 : DFP4_F32; }

// codes, dialect, exponent, rows, K
dfp4_tensor quantized(PyObject* const* a) {
    return dfp4_tensor{data(a[0]), data(a[1]), data(a[2]), number(a[3]), number(a[4])};
}

const at::Tensor& dense(PyObject* o) {
    const at::Tensor& x = tensor(o);
    if (x.scalar_type() != at::kBFloat16 || x.dim() != 2 || !x.is_cuda() || x.stride(1) != 1)
        fail(PyExc_AssertionError, "a bf16 matrix on the device, contiguous along its rows, is expected");
    return x;
}

template <class F>
PyObject* call(Py_ssize_t given, Py_ssize_t wanted, F&& f) {
    if (given != wanted) {
        PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
        return nullptr;
    }
    try {
        return f();
    } catch (const Failure&) {
    } catch (...) {
        // as torch.empty raises them: an exhausted device is a torch.OutOfMemoryError
        torch::translate_exception_to_python(std::current_exception());
    }
    return nullptr;
}

// quantize(x, block, mx) -> codes, dialect, exponent, rows, K
PyObject* quantize(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return call(n, 3, [&]() -> PyObject* {
        const at::Tensor& x = dense(a[0]);
        const int64_t block = number(a[1]), rows = x.size(0), K = x.size(1), per = block == 16 ? 16 : 32;
        const bool mx = a[2] == Py_True;
        const at::Device dev = x.device();
        at::Tensor codes = bytes(rows, K / 2, dev), dialect, exponent = bytes(rows, K / per, dev);
        if (!mx) dialect = bytes(rows, K / per, dev);
        const dfp4_tensor q{data(codes), mx ? nullptr : data(dialect), data(exponent), rows, K};
        const int64_t ld = rows > 1 ? x.stride(0) : K;
        if (mx) enqueue("mxfp4_quantize", p_mxfp4_quantize, data(x), rows, K, ld, q, stream());
        else if (block == 32) enqueue("dfp4_quantize", p_dfp4_quantize, data(x), rows, K, ld, q, stream());
        else enqueue("dfp4_quantize_block", p_dfp4_quantize_block, data(x), rows, K, ld, (int)block, q, stream());
        PyObject* d = mx ? Py_NewRef(Py_None) : THPVariable_Wrap(std::move(dialect));
        return Py_BuildValue("NNNLL", THPVariable_Wrap(std::move(codes)), d, THPVariable_Wrap(std::move(exponent)), (long long)rows, (long long)K);
    });
}

// dequantize(codes, dialect, exponent, rows, K, bf16, mx) -> y
PyObject* dequantize(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return call(n, 7, [&] {
        const dfp4_tensor q = quantized(a);
        const bool bf16 = a[5] == Py_True, mx = a[6] == Py_True;
        at::Tensor y = result({q.rows, q.K}, bf16, tensor(a[0]).device());
        enqueue(mx ? "mxfp4_dequantize" : "dfp4_dequantize", mx ? p_mxfp4_dequantize : p_dfp4_dequantize, q, data(y), dtype(bf16), q.K, stream());
        return THPVariable_Wrap(std::move(y));
    });
}

// gemm(a's five, w's five, bf16, mx) -> out
PyObject* gemm(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return call(n, 12, [&] {
        const dfp4_tensor A = quantized(a), W = quantized(a + 5);
        const bool bf16 = a[10] == Py_True, mx = a[11] == Py_True;
        const at::Device dev = tensor(a[0]).device();
        at::Tensor out = result({A.rows, W.rows}, bf16, dev), ws;
        const size_t need = p_dfp4_gemm_workspace_bytes(A.rows, W.rows, A.K);
        if (need > 0) ws = bytes((int64_t)need, dev);
        enqueue(mx ? "mxfp4_gemm" : "dfp4_gemm", mx ? p_mxfp4_gemm : p_dfp4_gemm, A, W, data(out), dtype(bf16), W.rows, need > 0 ? data(ws) : nullptr, need,
                stream());
        return THPVariable_Wrap(std::move(out));
    });
}

// gemm_batched(a's five, w's five, batch, M, N, bf16) -> out
PyObject* gemm_batched(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return call(n, 14, [&] {
        dfp4_tensor A = quantized(a), W = quantized(a + 5);
        const int64_t batch = number(a[10]), M = number(a[11]), N = number(a[12]);
        const bool bf16 = a[13] == Py_True;
        const at::Device dev = tensor(a[0]).device();
        A.rows = M;
        W.rows = N;
        at::Tensor out = result({batch, M, N}, bf16, dev), ws;
        const size_t need = p_dfp4_gemm_workspace_bytes(M, N, A.K) * (size_t)batch;
        if (need > 0) ws = bytes((int64_t)need, dev);
        enqueue("dfp4_gemm_batched", p_dfp4_gemm_batched, A, W, data(out), dtype(bf16), N, batch, M, N, M * N, need > 0 ? data(ws) : nullptr, need,
                stream());
        return THPVariable_Wrap(std::move(out));
    });
}

// gemm_prepare(five, weight, mx) -> buffer, or None where nothing is prepared
PyObject* gemm_prepare(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return call(n, 7, [&]() -> PyObject* {
        const dfp4_tensor q = quantized(a);
        const int weight = a[5] == Py_True ? 1 : 0;
        const size_t need = p_dfp4_gemm_prepared_bytes(q.rows, q.K, weight);
        if (need == 0) Py_RETURN_NONE;
        at::Tensor buf = bytes((int64_t)need, tensor(a[0]).device());
        enqueue("gemm_prepare", a[6] == Py_True ? p_mxfp4_gemm_prepare : p_dfp4_gemm_prepare, q, weight, data(buf), need, stream());
        return THPVariable_Wrap(std::move(buf));
    });
}

// gemm_prepared(a's five, its buffer, w's five, its buffer, bf16, mx) -> out
PyObject* gemm_prepared(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return call(n, 14, [&] {
        const dfp4_tensor A = quantized(a), W = quantized(a + 6);
        const bool bf16 = a[12] == Py_True, mx = a[13] == Py_True;
        const at::Device dev = tensor(a[0]).device();
        at::Tensor out = result({A.rows, W.rows}, bf16, dev), ws;
        const size_t need = p_dfp4_gemm_prepared_workspace_bytes(A.rows, W.rows, A.K);
        if (need > 0) ws = bytes((int64_t)need, dev);
        enqueue("gemm_prepared", mx ? p_mxfp4_gemm_prepared : p_dfp4_gemm_prepared, A, data(a[5]), W, data(a[11]), data(out), dtype(bf16), W.rows,
                need > 0 ? data(ws) : nullptr, need, stream());
        return THPVariable_Wrap(std::move(out));
    });
}

// quantize_native(x) -> buffer (x not empty)
PyObject* quantize_native(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return call(n, 1, [&] {
        const at::Tensor& x = dense(a[0]);
        const int64_t rows = x.size(0), K = x.size(1);
        at::Tensor buf = bytes((int64_t)p_dfp4_native_packed_bytes(rows, K), x.device());
        enqueue("dfp4_quantize_native", p_dfp4_quantize_native, data(x), rows, K, rows > 1 ? x.stride(0) : K, data(buf), (size_t)buf.numel(), stream());
        return THPVariable_Wrap(std::move(buf));
    });
}

// native_pack(five, mx) -> buffer
PyObject* native_pack(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return call(n, 6, [&] {
        const dfp4_tensor q = quantized(a);
        const int64_t need = (int64_t)p_dfp4_native_packed_bytes(q.rows, q.K);
        at::Tensor buf = bytes(need > 256 ? need : 256, tensor(a[0]).device());
        enqueue("native_pack", a[5] == Py_True ? p_mxfp4_native_pack : p_dfp4_native_pack, q, data(buf), (size_t)buf.numel(), stream());
        return THPVariable_Wrap(std::move(buf));
    });
}

// gemm_native_packed(a's buffer, M, w's buffer, N, K, bf16, mx) -> out
PyObject* gemm_native_packed(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return call(n, 7, [&] {
        const int64_t M = number(a[1]), N = number(a[3]), K = number(a[4]);
        const bool bf16 = a[5] == Py_True, mx = a[6] == Py_True;
        const at::Device dev = tensor(a[0]).device();
        at::Tensor out = result({M, N}, bf16, dev), ws;
        const size_t need = p_dfp4_gemm_native_splitk_bytes(M, N, K);
        if (need > 0) ws = bytes((int64_t)need, dev);
        enqueue("gemm_native_packed", mx ? p_mxfp4_gemm_native_packed : p_dfp4_gemm_native_packed, data(a[0]), M, data(a[2]), N, K, data(out), dtype(bf16), N,
                need > 0 ? data(ws) : nullptr, need, stream());
        return THPVariable_Wrap(std::move(out));
    });
}

// bind(path of libdfp4.so, exception class)
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return call(n, 2, [&]() -> PyObject* {
        const char* path = PyUnicode_AsUTF8(a[0]);
        if (!path) throw Failure{};
        void* lib = dlopen(path, RTLD_NOW | RTLD_LOCAL);
        if (!lib) fail(PyExc_OSError, dlerror());
#define DFP4_BIND(NAME)                                                          \
        p_##NAME = reinterpret_cast<decltype(&::NAME)>(dlsym(lib, #NAME));       \
        if (!p_##NAME) fail(PyExc_OSError, "libdfp4.so has no " #NAME);
        DFP4_FUNCTIONS(DFP4_BIND)
#undef DFP4_BIND
        Py_XSETREF(g_error, Py_NewRef(a[1]));
        Py_RETURN_NONE;
    });
}

#define DFP4_METHOD(NAME) {#NAME, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(NAME)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {DFP4_METHOD(bind), DFP4_METHOD(quantize), DFP4_METHOD(dequantize), DFP4_METHOD(gemm), DFP4_METHOD(gemm_batched),
                         DFP4_METHOD(gemm_prepare), DFP4_METHOD(gemm_prepared), DFP4_METHOD(quantize_native), DFP4_METHOD(native_pack),
                         DFP4_METHOD(gemm_native_packed), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() { return PyModule_Create(&module); }
