// CPython binding of the calls a decoding step makes (paper_2501_01144_amd/dfp4.py wraps the others with ctypes).
//
// At a few rows a pass is two kernels of 3 and 11 us; marshalled in Python (three tensor allocations through the
// argument parser, structs and pointers through ctypes, a workspace query) it took 25 us of host time and the GPU
// waited for the host.  Here the output tensors are allocated through ATen directly and the C ABI is called with the
// arguments read from the Python objects.
// BINDINGMEASURED
//
// Every function takes the stream as an integer, returns the C ABI's status, and does no checks of its own beyond
// what keeps it from misreading its arguments: the callers in dfp4.py assert what the C ABI cannot see.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/dfp4.h"

namespace {

const at::Tensor& tensor(PyObject* o) {
    TORCH_CHECK_TYPE(THPVariable_Check(o), "expected a tensor, got ", Py_TYPE(o)->tp_name);
    return THPVariable_Unpack(o);
}
// device pointer of a tensor; null for None and for an empty tensor
void* pointer(PyObject* o) {
    if (o == Py_None) return nullptr;
    const at::Tensor& t = tensor(o);
    return t.numel() > 0 ? t.data_ptr() : nullptr;
}
int64_t integer(PyObject* o) {
    const int64_t v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw python_error();
    return v;
}
void* stream(PyObject* o) { return reinterpret_cast<void*>(static_cast<uintptr_t>(integer(o))); }

struct Attr {                                            // an attribute, released at the end of the scope
    PyObject* o;
    Attr(PyObject* of, PyObject* name) : o(PyObject_GetAttr(of, name)) {
        if (!o) throw python_error();
    }
    ~Attr() { Py_DECREF(o); }
    Attr(const Attr&) = delete;
    Attr& operator=(const Attr&) = delete;
};
PyObject *s_codes, *s_dialect, *s_exponent, *s_rows, *s_K;

dfp4_tensor quantized(PyObject* q) {
    const Attr c(q, s_codes), d(q, s_dialect), e(q, s_exponent), r(q, s_rows), k(q, s_K);
    dfp4_tensor t{};
    t.codes = static_cast<uint8_t*>(pointer(c.o));
    t.dialect = static_cast<uint8_t*>(pointer(d.o));
    t.exponent = static_cast<uint8_t*>(pointer(e.o));
    t.rows = integer(r.o);
    t.K = integer(k.o);
    return t;
}
at::Tensor bytes(at::IntArrayRef size, const at::Device& device) {
    return at::empty(size, at::TensorOptions().dtype(at::kByte).device(device));
}
void want(Py_ssize_t n, Py_ssize_t expected) {
    TORCH_CHECK_TYPE(n == expected, "expected ", expected, " arguments, got ", n);
}
struct NoGil {                                           // the GIL is not held while the library launches
    PyThreadState* s = PyEval_SaveThread();
    ~NoGil() { PyEval_RestoreThread(s); }
};

// quantize(kind, x, stream) -> (status, codes, dialect | None, exponent); x: bf16 [rows, K], unit column stride
enum { kDfp4, kMxfp4, kDfp4T, kMxfp4T };
PyObject* quantize(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    want(n, 3);
    const int64_t kind = integer(a[0]);
    const at::Tensor& x = tensor(a[1]);
    const bool mx = kind == kMxfp4 || kind == kMxfp4T, transposed = kind >= kDfp4T;
    const int64_t rows = x.size(0), cols = x.size(1), ld = rows > 1 ? x.stride(0) : cols;
    const int64_t out_rows = transposed ? cols : rows, K = transposed ? rows : cols;
    at::Tensor codes = bytes({out_rows, K / 2}, x.device()), expo = bytes({out_rows, K / 32}, x.device()), dial;
    if (!mx) dial = bytes({out_rows, K / 32}, x.device());
    auto ptr = [](const at::Tensor& t) { return t.defined() && t.numel() > 0 ? static_cast<uint8_t*>(t.data_ptr()) : nullptr; };
    const dfp4_tensor q{ptr(codes), ptr(dial), ptr(expo), out_rows, K};
    const void* xp = x.numel() > 0 ? x.data_ptr() : nullptr;
    void* st = stream(a[2]);
    auto* call = kind == kDfp4 ? dfp4_quantize : kind == kMxfp4 ? mxfp4_quantize : kind == kDfp4T ? dfp4_quantize_t : mxfp4_quantize_t;
    int rc;
    {
        NoGil g;
        rc = call(xp, rows, cols, ld, q, st);
    }
    return Py_BuildValue("iNNN", rc, THPVariable_Wrap(std::move(codes)), mx ? Py_NewRef(Py_None) : THPVariable_Wrap(std::move(dial)),
                         THPVariable_Wrap(std::move(expo)));
    END_HANDLE_TH_ERRORS
}

// gemm_prepare(mx, q, weight, stream) -> (status, buffer | None)
PyObject* gemm_prepare(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    want(n, 4);
    const bool mx = integer(a[0]) != 0;
    const dfp4_tensor q = quantized(a[1]);
    const int weight = (int)integer(a[2]);
    void* st = stream(a[3]);
    const size_t need = dfp4_gemm_prepared_bytes(q.rows, q.K, weight);
    if (need == 0) return Py_BuildValue("iO", 0, Py_None);
    const Attr codes(a[1], s_codes);
    at::Tensor buf = bytes({(int64_t)need}, tensor(codes.o).device());
    int rc;
    {
        NoGil g;
        rc = (mx ? mxfp4_gemm_prepare : dfp4_gemm_prepare)(q, weight, buf.data_ptr(), need, st);
    }
    return Py_BuildValue("iN", rc, THPVariable_Wrap(std::move(buf)));
    END_HANDLE_TH_ERRORS
}

// The output's leading dimension and type, and a workspace of `need` bytes unless the caller brought one
struct Output {
    void* ptr;
    int dtype;
    int64_t ldc;
    at::Tensor own_ws;
    void* ws = nullptr;
    size_t ws_bytes = 0;
    Output(PyObject* out, int64_t M, int64_t N, PyObject* workspace, size_t need) {
        const at::Tensor& o = tensor(out);
        ptr = o.numel() > 0 ? o.data_ptr() : nullptr;
        dtype = o.scalar_type() == at::kFloat ? DFP4_F32 : DFP4_BF16;
        ldc = M > 1 ? o.stride(0) : N;
        if (workspace != Py_None) {
            ws = pointer(workspace);
            ws_bytes = (size_t)tensor(workspace).numel();
        } else if (need > 0) {
            own_ws = bytes({(int64_t)need}, o.device());
            ws = own_ws.data_ptr();
            ws_bytes = need;
        }
    }
};

// gemm(mx, a, w, out, workspace | None, stream) -> status
PyObject* gemm(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    want(n, 6);
    const bool mx = integer(a[0]) != 0;
    const dfp4_tensor A = quantized(a[1]), W = quantized(a[2]);
    const Output o(a[3], A.rows, W.rows, a[4], a[4] == Py_None ? dfp4_gemm_workspace_bytes(A.rows, W.rows, A.K) : 0);
    void* st = stream(a[5]);
    int rc;
    {
        NoGil g;
        rc = (mx ? mxfp4_gemm : dfp4_gemm)(A, W, o.ptr, o.dtype, o.ldc, o.ws, o.ws_bytes, st);
    }
    return PyLong_FromLong(rc);
    END_HANDLE_TH_ERRORS
}

// gemm_prepared(mx, a, a_buf, w, w_buf, out, workspace | None, stream) -> status
PyObject* gemm_prepared(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    want(n, 8);
    const bool mx = integer(a[0]) != 0;
    const dfp4_tensor A = quantized(a[1]), W = quantized(a[3]);
    void *ap = pointer(a[2]), *wp = pointer(a[4]);
    const Output o(a[5], A.rows, W.rows, a[6], a[6] == Py_None ? dfp4_gemm_prepared_workspace_bytes(A.rows, W.rows, A.K) : 0);
    void* st = stream(a[7]);
    int rc;
    {
        NoGil g;
        rc = (mx ? mxfp4_gemm_prepared : dfp4_gemm_prepared)(A, ap, W, wp, o.ptr, o.dtype, o.ldc, o.ws, o.ws_bytes, st);
    }
    return PyLong_FromLong(rc);
    END_HANDLE_TH_ERRORS
}

// quantize_native(x, buf, stream) -> status; x: bf16 [rows, K], unit column stride
PyObject* quantize_native(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    want(n, 3);
    const at::Tensor &x = tensor(a[0]), &buf = tensor(a[1]);
    const int64_t rows = x.size(0), K = x.size(1), ld = rows > 1 ? x.stride(0) : K;
    const void* xp = x.numel() > 0 ? x.data_ptr() : nullptr;
    void *bp = buf.numel() > 0 ? buf.data_ptr() : nullptr, *st = stream(a[2]);
    const size_t nb = (size_t)buf.numel();
    int rc;
    {
        NoGil g;
        rc = dfp4_quantize_native(xp, rows, K, ld, bp, nb, st);
    }
    return PyLong_FromLong(rc);
    END_HANDLE_TH_ERRORS
}

// gemm_native_packed(mx, a_buf, M, w_buf, N, K, out, workspace | None, stream) -> status
PyObject* gemm_native_packed(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    want(n, 9);
    const bool mx = integer(a[0]) != 0;
    const int64_t M = integer(a[2]), N = integer(a[4]), K = integer(a[5]);
    void *ap = pointer(a[1]), *wp = pointer(a[3]);
    const Output o(a[6], M, N, a[7], a[7] == Py_None ? dfp4_gemm_native_splitk_bytes(M, N, K) : 0);
    void* st = stream(a[8]);
    int rc;
    {
        NoGil g;
        rc = (mx ? mxfp4_gemm_native_packed : dfp4_gemm_native_packed)(ap, M, wp, N, K, o.ptr, o.dtype, o.ldc, o.ws, o.ws_bytes, st);
    }
    return PyLong_FromLong(rc);
    END_HANDLE_TH_ERRORS
}

PyMethodDef methods[] = {
    {"quantize", (PyCFunction)(void (*)())quantize, METH_FASTCALL, nullptr},
    {"gemm_prepare", (PyCFunction)(void (*)())gemm_prepare, METH_FASTCALL, nullptr},
    {"gemm", (PyCFunction)(void (*)())gemm, METH_FASTCALL, nullptr},
    {"gemm_prepared", (PyCFunction)(void (*)())gemm_prepared, METH_FASTCALL, nullptr},
    {"quantize_native", (PyCFunction)(void (*)())quantize_native, METH_FASTCALL, nullptr},
    {"gemm_native_packed", (PyCFunction)(void (*)())gemm_native_packed, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() {
    s_codes = PyUnicode_InternFromString("codes");
    s_dialect = PyUnicode_InternFromString("dialect");
    s_exponent = PyUnicode_InternFromString("exponent");
    s_rows = PyUnicode_InternFromString("rows");
    s_K = PyUnicode_InternFromString("K");
    return PyModule_Create(&module);
}
