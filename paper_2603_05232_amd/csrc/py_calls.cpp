// The calls of a model's forward pass (quantisation, sparse GEMMs) as CPython functions: argument reading, output
// allocation and the C call without going through ctypes and torch's Python layer.  Layers of few tokens are bound by the time
// between launches, most of which was spent there (quantisation + GEMM of 16 x 512 x 512: see binding.py).
//
// Each function does plain calls only: exact torch.Tensor arguments on the GPU, exact ints, no active function or dispatch
// mode, and arguments that the C entry point accepts.  For anything else it returns None and the caller's general path does the
// call over, which is where arguments are refused and errors raised: the C entry points check their arguments before they launch
// anything.  A launch that failed is no argument to refuse: SS_ERR_HIP raises here, since a second attempt would launch
// again and find the runtime's error cleared.
//
// The module is not linked against libslidesparse.so: the binding hands it the addresses of the library that it has loaded by path.
// By name, the loader would give a second copy of the package in the process the first copy's library.
#include <Python.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <limits.h>
#include <string.h>
#include "slidesparse.h"

namespace {

struct Library {
    decltype(&::slide_lifted_ld) lifted_ld;
    decltype(&::act_lift_quant) lift_quant;
    decltype(&::slide_sparse_gemm_ws) sparse_gemm;
    decltype(&::slide_sparse_gemm_fused_ws) sparse_gemm_fused;
} lib;                                                // zeros until bind()
PyObject* error_type = nullptr;                       // SlideSparseError(status, where)

// the interpreter lock is given up while memory is allocated and kernels are launched (either may wait for the GPU)
struct Unlocked {
    PyThreadState* state = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(state); }
};

bool plain(PyObject* o)
{
    if (!THPVariable_CheckExact(o)) return false;
    constexpr c10::DispatchKeySet wrapped({c10::DispatchKey::Python, c10::DispatchKey::PythonTLSSnapshot, c10::DispatchKey::FuncTorchBatched,
                                           c10::DispatchKey::FuncTorchGradWrapper, c10::DispatchKey::Functionalize, c10::DispatchKey::Sparse,
                                           c10::DispatchKey::SparseCsr});
    const at::Tensor& t = THPVariable_Unpack(o);
    return t.defined() && t.has_storage() && !t.key_set().has_any(wrapped);
}
bool plain_or_none(PyObject* o) { return o == Py_None || plain(o); }
void* address(PyObject* o) { return o == Py_None ? nullptr : THPVariable_Unpack(o).data_ptr(); }

bool integer(PyObject* o, int64_t lo, int64_t hi, int64_t& v)
{
    if (!PyLong_CheckExact(o)) return false;
    int over = 0;
    const long long x = PyLong_AsLongLongAndOverflow(o, &over);
    if (over || x < lo || x > hi) return false;
    v = x;
    return true;
}

struct Type { ss_dtype code; at::ScalarType storage; bool scaled; };
bool operand_type(PyObject* o, Type& t)
{
    if (!PyUnicode_CheckExact(o)) return false;
    if (PyUnicode_CompareWithASCIIString(o, "i8") == 0) t = {SS_I8, at::kChar, true};
    else if (PyUnicode_CompareWithASCIIString(o, "fp8") == 0) t = {SS_FP8_E4M3, at::kByte, true};
    else if (PyUnicode_CompareWithASCIIString(o, "bf16") == 0) t = {SS_BF16, at::kBFloat16, false};
    else if (PyUnicode_CompareWithASCIIString(o, "fp16") == 0) t = {SS_FP16, at::kHalf, false};
    else return false;
    return true;
}

bool modes_active() { return c10::impl::TorchDispatchModeTLS::any_modes_set() || at::impl::torch_function_mode_enabled(); }
void* current_stream() { return c10::hip::getCurrentHIPStream().stream(); }

// what a function returns for a status other than SS_OK
PyObject* refused(ss_status st, const char* where)
{
    if (st != SS_ERR_HIP) Py_RETURN_NONE;
    if (PyObject* e = PyObject_CallFunction(error_type, "is", (int)st, where)) {
        PyErr_SetObject(error_type, e);
        Py_DECREF(e);
    }
    return nullptr;
}

// act_lift_quant(X, N, dtype, out, s_x)
PyObject* py_act_lift_quant(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    int64_t N;
    Type t;
    if (!lib.lift_quant || n != 5 || !plain(a[0]) || !integer(a[1], INT_MIN, INT_MAX, N) || !operand_type(a[2], t) || !plain_or_none(a[3]) || !plain_or_none(a[4]) || modes_active()) Py_RETURN_NONE;
    const at::Tensor& X = THPVariable_Unpack(a[0]);
    if (!X.is_cuda() || X.dim() != 2 || X.stride(1) != 1 || (X.scalar_type() != at::kFloat && X.scalar_type() != at::kBFloat16)) Py_RETURN_NONE;
    const int64_t M = X.size(0), K = X.size(1), width = lib.lifted_ld(K, (int)N, t.code);
    if (width < 0) Py_RETURN_NONE;
    at::Tensor out, s_x;
    void *out_ptr = address(a[3]), *s_x_ptr = address(a[4]);
    ss_status st;
    {
        Unlocked u;
        if (a[3] == Py_None) { out = at::empty({M, width}, X.options().dtype(t.storage)); out_ptr = out.data_ptr(); }
        if (a[4] == Py_None && t.scaled) { s_x = at::empty({M}, X.options().dtype(at::kFloat)); s_x_ptr = s_x.data_ptr(); }
        st = lib.lift_quant(X.data_ptr(), X.scalar_type() == at::kFloat ? SS_IN_F32 : SS_IN_BF16, M, K, M > 1 ? X.stride(0) : K, (int)N, t.code, out_ptr,
                            static_cast<float*>(s_x_ptr), current_stream());
    }
    if (st != SS_OK) return refused(st, "act_lift_quant");
    PyObject* po = out.defined() ? THPVariable_Wrap(std::move(out)) : Py_NewRef(a[3]);
    PyObject* ps = s_x.defined() ? THPVariable_Wrap(std::move(s_x)) : Py_NewRef(a[4]);
    PyObject* r = po && ps ? PyTuple_Pack(2, po, ps) : nullptr;
    Py_XDECREF(po);
    Py_XDECREF(ps);
    return r;
    END_HANDLE_TH_ERRORS
}

// The operands common to both GEMMs: a = X, s_x, w_vals, w_meta, s_w; `out` and `workspace` may be None
struct Out { at::Tensor made; void* ptr; int64_t ld; };
bool gemm_operands(PyObject* const* a, PyObject* out, PyObject* workspace)
{
    return plain(a[0]) && plain_or_none(a[1]) && plain_or_none(a[2]) && plain_or_none(a[3]) && plain_or_none(a[4]) && plain_or_none(out) &&
           (out == Py_None || THPVariable_Unpack(out).dim() == 2) && plain_or_none(workspace) && !modes_active();
}
Out output(PyObject* out, const at::Tensor& X, int64_t M, int64_t O)
{
    if (out != Py_None) return {at::Tensor(), THPVariable_Unpack(out).data_ptr(), THPVariable_Unpack(out).stride(0)};
    Out r{at::empty({M, O}, X.options().dtype(at::kBFloat16)), nullptr, 0};
    r.ptr = r.made.data_ptr();
    r.ld = r.made.stride(0);
    return r;
}
PyObject* result(Out& r, PyObject* out) { return r.made.defined() ? THPVariable_Wrap(std::move(r.made)) : Py_NewRef(out); }

// slide_sparse_gemm(X_lifted, s_x, w_vals, w_meta, s_w, O, dtype, out, workspace)
PyObject* py_slide_sparse_gemm(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    int64_t O;
    Type t;
    if (!lib.sparse_gemm || n != 9 || !gemm_operands(a, a[7], a[8]) || !integer(a[5], 0, INT64_MAX, O) || !operand_type(a[6], t)) Py_RETURN_NONE;
    const at::Tensor& X = THPVariable_Unpack(a[0]);
    if (!X.is_cuda() || X.dim() != 2 || !X.is_contiguous()) Py_RETURN_NONE;
    void* const ws = address(a[8]);
    const size_t ws_bytes = a[8] == Py_None ? 0 : THPVariable_Unpack(a[8]).nbytes();
    const void *s_x = address(a[1]), *wv = address(a[2]), *wm = address(a[3]), *s_w = address(a[4]);
    Out y;
    ss_status st;
    {
        Unlocked u;
        y = output(a[7], X, X.size(0), O);
        st = lib.sparse_gemm(X.data_ptr(), static_cast<const float*>(s_x), wv, wm, static_cast<const float*>(s_w), X.size(0), O, X.size(1), t.code, y.ptr, y.ld, ws, ws_bytes,
                                  current_stream());
    }
    if (st != SS_OK) return refused(st, a[8] == Py_None ? "slide_sparse_gemm" : "slide_sparse_gemm_ws");
    return result(y, a[7]);
    END_HANDLE_TH_ERRORS
}

// slide_sparse_gemm_fused(Xq, s_x, w_vals, w_meta, s_w, O, K, N, dtype, out, workspace)
PyObject* py_slide_sparse_gemm_fused(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    int64_t O, K, N;
    Type t;
    if (!lib.sparse_gemm_fused || n != 11 || !gemm_operands(a, a[9], a[10]) || !integer(a[5], 0, INT64_MAX, O) || !integer(a[6], 0, INT64_MAX, K) || !integer(a[7], INT_MIN, INT_MAX, N) ||
        !operand_type(a[8], t))
        Py_RETURN_NONE;
    const at::Tensor& X = THPVariable_Unpack(a[0]);
    if (!X.is_cuda() || X.dim() != 2 || X.stride(1) != 1 || X.size(1) < K) Py_RETURN_NONE;
    const int64_t M = X.size(0);
    void* const ws = address(a[10]);
    const size_t ws_bytes = a[10] == Py_None ? 0 : (size_t)THPVariable_Unpack(a[10]).numel();
    const void *s_x = address(a[1]), *wv = address(a[2]), *wm = address(a[3]), *s_w = address(a[4]);
    Out y;
    ss_status st;
    {
        Unlocked u;
        y = output(a[9], X, M, O);
        st = lib.sparse_gemm_fused(X.data_ptr(), static_cast<const float*>(s_x), wv, wm, static_cast<const float*>(s_w), M, O, K, M > 1 ? X.stride(0) : X.size(1), (int)N,
                                        t.code, y.ptr, y.ld, ws, ws_bytes, current_stream());
    }
    if (st != SS_OK) return refused(st, a[10] == Py_None ? "slide_sparse_gemm_fused" : "slide_sparse_gemm_fused_ws");
    return result(y, a[9]);
    END_HANDLE_TH_ERRORS
}

// bind(SlideSparseError, slide_lifted_ld, act_lift_quant, slide_sparse_gemm_ws, slide_sparse_gemm_fused_ws), the last four as
// addresses; library() tells these
PyObject* py_bind(PyObject*, PyObject* args)
{
    PyObject* error;
    unsigned long long f[4];
    if (!PyArg_ParseTuple(args, "OKKKK", &error, &f[0], &f[1], &f[2], &f[3])) return nullptr;
    lib = {reinterpret_cast<decltype(lib.lifted_ld)>(f[0]), reinterpret_cast<decltype(lib.lift_quant)>(f[1]), reinterpret_cast<decltype(lib.sparse_gemm)>(f[2]),
           reinterpret_cast<decltype(lib.sparse_gemm_fused)>(f[3])};
    Py_INCREF(error);
    Py_XDECREF(error_type);
    error_type = error;
    Py_RETURN_NONE;
}
PyObject* py_library(PyObject*, PyObject*)
{
    return Py_BuildValue("KKKK", reinterpret_cast<unsigned long long>(lib.lifted_ld), reinterpret_cast<unsigned long long>(lib.lift_quant),
                         reinterpret_cast<unsigned long long>(lib.sparse_gemm), reinterpret_cast<unsigned long long>(lib.sparse_gemm_fused));
}

#define SS_PY(f) reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(f)), METH_FASTCALL
PyMethodDef methods[] = {{"act_lift_quant", SS_PY(py_act_lift_quant), nullptr},
                         {"slide_sparse_gemm", SS_PY(py_slide_sparse_gemm), nullptr},
                         {"slide_sparse_gemm_fused", SS_PY(py_slide_sparse_gemm_fused), nullptr},
                         {"bind", py_bind, METH_VARARGS, nullptr},
                         {"library", py_library, METH_NOARGS, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls(void)
{
    PyObject* m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "torch_version", SS_TORCH_VERSION) < 0) Py_CLEAR(m);      // torch's C++ interface is another one in each version
    return m;
}
