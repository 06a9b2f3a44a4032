// tsg_calls.cpp -- the plain calls of tsmttsm and tsmm on torch tensors, native.
//
// A call on a few thousand rows is bound by the host: of 13 us in Python
// (10007 x 4 and 4 doubles, calls in a row) the library took 4.5, the launch
// included, and the rest went into shapes, strides and pointers, the device
// context, the stream and the marshalling of 15 arguments.  Through these
// functions the whole call takes 4.7 us; an update of 10007 x 4 by 16 went from
// 11.2 to 5.3, now its kernel's time.  They take dense tensors on the current
// device and answer NotImplemented for everything else, before any effect:
// tensor subclasses, wrappers and modes, other devices, empty matrices,
// arguments that are wrong.  The Python functions then take the call and raise
// what there is to raise.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>

#include <cstring>

#include "tsgemm.h"

namespace {

decltype(&tsg_tsmttsm) g_tsmttsm = nullptr;
decltype(&tsg_tsmm_op) g_tsmm_op = nullptr;

PyObject* not_here() { Py_RETURN_NOTIMPLEMENTED; }

// The tensor of a plain, dense, non-empty matrix with unit column stride on
// device `dev` (-1: any), or null.
const at::Tensor* matrix(PyObject* o, int dev)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    using K = c10::DispatchKey;
    static const c10::DispatchKeySet plain{K::CUDA,        K::AutogradCUDA, K::AutocastCUDA, K::ADInplaceOrView,
                                           K::AutogradOther};
    if ((t.key_set().raw_repr() & ~plain.raw_repr()) || t.layout() != at::kStrided || t.dim() != 2 || !t.is_cuda()) return nullptr;
    if (t.size(0) == 0 || t.size(1) == 0 || (t.size(1) > 1 && t.stride(1) != 1)) return nullptr;
    return dev < 0 || t.get_device() == dev ? &t : nullptr;
}

int64_t ld(const at::Tensor& t)
{
    return t.size(0) > 1 ? t.stride(0) : t.size(1) > t.stride(0) ? t.size(1) : t.stride(0);
}

// Storage / arithmetic type of a call, and the type of its small matrix.
bool types(at::ScalarType s, PyObject* acc, tsg_dtype* dt, at::ScalarType* small)
{
    if (!PyUnicode_CheckExact(acc)) return false;
    const bool f32 = PyUnicode_CompareWithASCIIString(acc, "f32") == 0;
    if (!f32 && PyUnicode_CompareWithASCIIString(acc, "f64") != 0) return false;
    switch (s) {
    case at::kDouble: *dt = TSG_R64; break;
    case at::kComplexDouble: *dt = TSG_C128; break;
    case at::kFloat: *dt = f32 ? TSG_R32_ACC32 : TSG_R32; break;
    case at::kComplexFloat: *dt = f32 ? TSG_C64_ACC32 : TSG_C64; break;
    default: return false;
    }
    if (f32 && (*dt == TSG_R64 || *dt == TSG_C128)) return false;
    *small = at::isComplexType(s) ? at::kComplexDouble : at::kDouble;
    return true;
}

// No mode or transform sees the calls of this thread.
bool no_modes()
{
    if (c10::impl::dispatch_mode_enabled() || at::impl::torch_function_mode_enabled()) return false;
    return !(c10::impl::tls_local_dispatch_key_set().included_.raw_repr() & ~c10::default_included_set.raw_repr());
}

// -1, or the operation 'N', 'T', 'C' as the library's number (of `known`).
int operation(PyObject* o, const char* known)
{
    if (!PyUnicode_CheckExact(o) || PyUnicode_GetLength(o) != 1) return -1;
    const Py_UCS4 c = PyUnicode_ReadChar(o, 0);
    if (c > 127 || !strchr(known, (int)c)) return -1;
    return c == 'N' ? TSG_OP_N : c == 'T' ? TSG_OP_T : TSG_OP_C;
}

bool number(PyObject* o, double* out)
{
    if (PyFloat_CheckExact(o)) *out = PyFloat_AS_DOUBLE(o);
    else return false;
    return true;
}

// tsmttsm(A, B, op, out, acc): the result, a status to raise, or NotImplemented
PyObject* tsmttsm(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 5 || !g_tsmttsm) return not_here();
    const at::Tensor* A = matrix(args[0], -1);
    const at::Tensor* B = A ? matrix(args[1], A->get_device()) : nullptr;
    const int op = operation(args[2], "TC");
    tsg_dtype dt;
    at::ScalarType small;
    if (!B || op < 0 || !types(A->scalar_type(), args[4], &dt, &small) || B->scalar_type() != A->scalar_type() ||
        B->size(0) != A->size(0) || A->size(1) > 64 || B->size(1) > 64 || c10::hip::current_device() != A->get_device() || !no_modes())
        return not_here();
    const int64_t K = A->size(0), M = A->size(1), N = B->size(1);
    at::Tensor fresh;
    const at::Tensor* out;
    if (args[3] == Py_None) {
        fresh = at::empty({M, N}, A->options().dtype(small).requires_grad(false));
        out = &fresh;
    } else {
        out = matrix(args[3], A->get_device());
        if (!out || out->size(0) != M || out->size(1) != N || out->scalar_type() != small) return not_here();
    }
    const void *a = A->data_ptr(), *b = B->data_ptr();
    void* c = out->data_ptr();
    const int64_t la = ld(*A), lb = ld(*B), lc = ld(*out);
    void* stream = c10::hip::getCurrentHIPStream(A->get_device()).stream();
    tsg_status s;
    Py_BEGIN_ALLOW_THREADS
    s = g_tsmttsm(dt, (tsg_op)op, K, (int32_t)M, (int32_t)N, a, la, b, lb, c, lc, stream);
    Py_END_ALLOW_THREADS
    if (s != TSG_OK) return PyLong_FromLong(s);
    if (args[3] == Py_None) return THPVariable_Wrap(fresh);
    Py_INCREF(args[3]);
    return args[3];
    END_HANDLE_TH_ERRORS
}

// tsmm(A, C, out, alpha, beta, conjA, opC, acc)
PyObject* tsmm(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 8 || !g_tsmm_op) return not_here();
    const at::Tensor* A = matrix(args[0], -1);
    const at::Tensor* C = A ? matrix(args[1], A->get_device()) : nullptr;
    const int op = operation(args[6], "NTC");
    double alpha, beta;
    tsg_dtype dt;
    at::ScalarType small;
    if (!C || op < 0 || !number(args[3], &alpha) || !number(args[4], &beta) || !PyBool_Check(args[5]) ||
        !types(A->scalar_type(), args[7], &dt, &small) || C->scalar_type() != small ||
        c10::hip::current_device() != A->get_device() || !no_modes())
        return not_here();
    const int64_t K = A->size(0), M = A->size(1);
    const int64_t Mc = op == TSG_OP_N ? C->size(0) : C->size(1), N = op == TSG_OP_N ? C->size(1) : C->size(0);
    if (Mc != M || M > 64 || N > 64) return not_here();
    at::Tensor fresh;
    const at::Tensor* out;
    if (args[2] == Py_None) {
        if (beta != 0.0) return not_here();
        fresh = at::empty({K, N}, A->options().requires_grad(false));
        out = &fresh;
    } else {
        out = matrix(args[2], A->get_device());
        if (!out || out->size(0) != K || out->size(1) != N || out->scalar_type() != A->scalar_type()) return not_here();
    }
    const void *a = A->data_ptr(), *c = C->data_ptr();
    void* b = out->data_ptr();
    const int64_t la = ld(*A), lc = ld(*C), lb = ld(*out);
    void* stream = c10::hip::getCurrentHIPStream(A->get_device()).stream();
    tsg_status s;
    Py_BEGIN_ALLOW_THREADS
    s = g_tsmm_op(dt, args[5] == Py_True, (tsg_op)op, K, (int32_t)M, (int32_t)N, a, la, c, lc, b, lb, alpha, beta, stream);
    Py_END_ALLOW_THREADS
    if (s != TSG_OK) return PyLong_FromLong(s);
    if (args[2] == Py_None) return THPVariable_Wrap(fresh);
    Py_INCREF(args[2]);
    return args[2];
    END_HANDLE_TH_ERRORS
}

// bind(tsmttsm, tsmm_op): addresses of the loaded library's entry points
PyObject* bind(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    if (n != 2) return not_here();
    void *a = PyLong_AsVoidPtr(args[0]), *b = PyLong_AsVoidPtr(args[1]);
    if (PyErr_Occurred()) return nullptr;
    g_tsmttsm = reinterpret_cast<decltype(g_tsmttsm)>(a);
    g_tsmm_op = reinterpret_cast<decltype(g_tsmm_op)>(b);
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"tsmttsm", (PyCFunction)(void (*)(void))tsmttsm, METH_FASTCALL, nullptr},
    {"tsmm", (PyCFunction)(void (*)(void))tsmm, METH_FASTCALL, nullptr},
    {"bind", (PyCFunction)(void (*)(void))bind, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__calls()
{
    PyObject* m = PyModule_Create(&module);
    // what it was built for: another torch's tensors need not look alike
    if (m && PyModule_AddStringConstant(m, "torch_version", TSG_TORCH_VERSION) < 0) Py_CLEAR(m);
    return m;
}
