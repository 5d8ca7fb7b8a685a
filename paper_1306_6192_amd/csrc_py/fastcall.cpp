// Native call path of the Python layer's small entry points.
//
// A product of a few microseconds is bound by its caller: the checks, the
// output allocation, the stream query and the argument structs of the Python
// layer took 10 us a call (64^3 FP32: 12.1 us a pass, now 4.9), the launch 3.
// These functions do the
// same steps on the tensors' C++ side and call the same C-ABI entry points.
//
// They take a call only where every check of the Python layer would pass on
// plain strided device tensors; for anything else -- another layout, type,
// shape, tensor subclass, an active torch-function or dispatch mode, a
// functorch wrapper -- they return None before doing anything and the Python
// layer handles it (and raises its own errors).  On an error status of the
// library they return the status, which the Python layer raises.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/Exceptions.h>

#include "mi355gemm.h"

namespace {

typedef int (*PlainFn)(const gemm_problem_t *, void *);
typedef int (*SameTypeF64Fn)(int64_t, int64_t, int64_t, const double *, int64_t, const double *, int64_t, double *,
                             int64_t, void *);
typedef int (*SameTypeC32Fn)(int64_t, int64_t, int64_t, const float *, int64_t, const float *, int64_t, float *,
                             int64_t, void *);
typedef int (*ConvertFn)(const float *, int64_t, int32_t, void *, void *);
typedef int (*QuantizeFn)(const float *, int64_t, uint8_t *, float *, void *);

// Entry points of the library the Python layer has loaded (bind()).
PlainFn g_plain = nullptr;
SameTypeF64Fn g_f64 = nullptr;
SameTypeC32Fn g_c32 = nullptr;
ConvertFn g_convert = nullptr;
QuantizeFn g_quantize = nullptr;

bool modes_active() {
    return at::impl::torch_function_mode_enabled() || c10::impl::TorchDispatchModeTLS::any_modes_set();
}

// The tensor of a plain device tensor object (exactly torch.Tensor, strided,
// no dispatch beyond its device and autograd), or null.
const at::Tensor *plain_tensor(PyObject *o) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined()) return nullptr;
    static const c10::DispatchKeySet allowed =
        c10::DispatchKeySet({c10::DispatchKey::CUDA, c10::DispatchKey::ADInplaceOrView}) |
        c10::DispatchKeySet({c10::DispatchKey::AutogradCUDA, c10::DispatchKey::AutocastCUDA});
    if (!t.is_cuda() || t.layout() != c10::kStrided || !allowed.has_all(t.key_set())) return nullptr;
    return &t;
}

// The mode argument: exactly an int that names one (no error is left behind by
// one that does not fit).
bool mode_arg(PyObject *o, int *mode) {
    if (!PyLong_CheckExact(o)) return false;
    int over = 0;
    const long v = PyLong_AsLongAndOverflow(o, &over);
    if (over || v < 0 || v >= GEMM_NUM_MODES) return false;
    *mode = (int)v;
    return true;
}

// A row-major matrix as the Python layer accepts it.
bool matrix(const at::Tensor &t) {
    return t.dim() == 2 && !(t.size(0) > 0 && t.size(1) > 1 && t.stride(1) != 1);
}

int64_t leading(const at::Tensor &t) {
    const int64_t ld = t.size(0) > 1 ? t.stride(0) : t.size(1);
    return ld > 1 ? ld : 1;
}

bool type_ok(c10::ScalarType t, int mode) {
    using S = c10::ScalarType;
    switch (mode) {
        case GEMM_MODE_F32:
        case GEMM_MODE_F32_SPLIT_BF16X3: return t == S::Float;
        case GEMM_MODE_BF16: return t == S::BFloat16 || t == S::Short || t == S::UInt16;
        case GEMM_MODE_F16: return t == S::Half || t == S::Short || t == S::UInt16;
        case GEMM_MODE_F8E4M3: return t == S::Float8_e4m3fn || t == S::Byte || t == S::Char;
        default: return false;
    }
}

// The current stream of the current device.
void *current_stream() {
    return c10::hip::getCurrentHIPStream().stream();
}

const void *ptr(const at::Tensor &t) { return t.numel() ? t.data_ptr() : nullptr; }

// A fresh output, or `o`'s tensor where it fits; undefined: not for this path.
at::Tensor output(PyObject *o, const at::Tensor &like, int64_t m, int64_t n, c10::ScalarType type) {
    if (o == Py_None) return at::empty({m, n}, like.options().dtype(type).requires_grad(false));
    const at::Tensor *t = plain_tensor(o);
    if (!t || !matrix(*t) || t->scalar_type() != type || t->size(0) != m || t->size(1) != n) return at::Tensor();
    return *t;
}

PyObject *result(int rc, PyObject *given, const at::Tensor &out) {
    if (rc < 0) return PyLong_FromLong(rc);
    if (given != Py_None) {
        Py_INCREF(given);
        return given;
    }
    return THPVariable_Wrap(out);
}

// gemm(A, B, out, mode, scale_a, scale_b)
PyObject *fast_gemm(PyObject *, PyObject *const *args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    if (nargs != 6 || !g_plain || modes_active()) Py_RETURN_NONE;
    int mode = 0;
    if (!mode_arg(args[3], &mode) || !PyFloat_CheckExact(args[4]) || !PyFloat_CheckExact(args[5])) Py_RETURN_NONE;
    const at::Tensor *A = plain_tensor(args[0]), *B = plain_tensor(args[1]);
    if (!A || !B || !matrix(*A) || !matrix(*B) || !type_ok(A->scalar_type(), mode) ||
        !type_ok(B->scalar_type(), mode) || A->size(1) != B->size(0))
        Py_RETURN_NONE;
    const at::Tensor C = output(args[2], *A, A->size(0), B->size(1), c10::ScalarType::Float);
    if (!C.defined()) Py_RETURN_NONE;
    gemm_problem_t p;
    p.mode = mode;
    p.flags = 0;
    p.m = A->size(0);
    p.n = B->size(1);
    p.k = A->size(1);
    p.A = ptr(*A);
    p.lda = leading(*A);
    p.B = ptr(*B);
    p.ldb = leading(*B);
    p.C = (float *)ptr(C);
    p.ldc = leading(C);
    p.scale_a = (float)PyFloat_AS_DOUBLE(args[4]);
    p.scale_b = (float)PyFloat_AS_DOUBLE(args[5]);
    void *s = current_stream();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = g_plain(&p, s);
    Py_END_ALLOW_THREADS
    return result(rc, args[2], C);
    END_HANDLE_TH_ERRORS
}

// gemm_same(A, B, out): binary64 or complex float, by A's type
PyObject *fast_same(PyObject *, PyObject *const *args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    if (nargs != 3 || !g_f64 || !g_c32 || modes_active()) Py_RETURN_NONE;
    const at::Tensor *A = plain_tensor(args[0]), *B = plain_tensor(args[1]);
    if (!A || !B || !matrix(*A) || !matrix(*B) || A->scalar_type() != B->scalar_type() || A->size(1) != B->size(0))
        Py_RETURN_NONE;
    const bool f64 = A->scalar_type() == c10::ScalarType::Double;
    if (!f64 && A->scalar_type() != c10::ScalarType::ComplexFloat) Py_RETURN_NONE;
    const int64_t m = A->size(0), n = B->size(1), k = A->size(1);
    const at::Tensor C = output(args[2], *A, m, n, A->scalar_type());
    if (!C.defined() || A->is_conj() || B->is_conj() || C.is_conj()) Py_RETURN_NONE;
    void *s = current_stream();
    const int64_t la = leading(*A), lb = leading(*B), lc = leading(C);
    const void *a = ptr(*A), *b = ptr(*B), *c = ptr(C);
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f64 ? g_f64(m, n, k, (const double *)a, la, (const double *)b, lb, (double *)c, lc, s)
             : g_c32(m, n, k, (const float *)a, la, (const float *)b, lb, (float *)c, lc, s);
    Py_END_ALLOW_THREADS
    return result(rc, args[2], C);
    END_HANDLE_TH_ERRORS
}

// convert(x, mode)
PyObject *fast_convert(PyObject *, PyObject *const *args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    int mode = 0;
    if (nargs != 2 || !g_convert || modes_active() || !mode_arg(args[1], &mode)) Py_RETURN_NONE;
    const at::Tensor *x = plain_tensor(args[0]);
    if (!x || x->scalar_type() != c10::ScalarType::Float || !x->is_contiguous() ||
        (mode != GEMM_MODE_BF16 && mode != GEMM_MODE_F16))
        Py_RETURN_NONE;
    const at::Tensor out = at::empty(
        x->sizes(), x->options()
                        .dtype(mode == GEMM_MODE_BF16 ? c10::ScalarType::BFloat16 : c10::ScalarType::Half)
                        .requires_grad(false));
    void *s = current_stream();
    const void *src = ptr(*x), *dst = ptr(out);
    const int64_t count = x->numel();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = g_convert((const float *)src, count, mode, (void *)dst, s);
    Py_END_ALLOW_THREADS
    return result(rc, Py_None, out);
    END_HANDLE_TH_ERRORS
}

// quantize(x) -> (codes, scale)
PyObject *fast_quantize(PyObject *, PyObject *const *args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    if (nargs != 1 || !g_quantize || modes_active()) Py_RETURN_NONE;
    const at::Tensor *x = plain_tensor(args[0]);
    if (!x || x->scalar_type() != c10::ScalarType::Float || !x->is_contiguous()) Py_RETURN_NONE;
    const at::TensorOptions o = x->options().requires_grad(false);
    const at::Tensor q = at::empty(x->sizes(), o.dtype(c10::ScalarType::Byte));
    const at::Tensor scale = at::empty({1}, o);
    void *s = current_stream();
    const void *src = ptr(*x), *dst = ptr(q);
    float *sp = scale.data_ptr<float>();
    const int64_t count = x->numel();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = g_quantize((const float *)src, count, (uint8_t *)dst, sp, s);
    Py_END_ALLOW_THREADS
    if (rc < 0) return PyLong_FromLong(rc);
    PyObject *a = THPVariable_Wrap(q), *b = THPVariable_Wrap(scale);
    PyObject *t = a && b ? PyTuple_Pack(2, a, b) : nullptr;
    Py_XDECREF(a);
    Py_XDECREF(b);
    return t;
    END_HANDLE_TH_ERRORS
}

// bind(gemm_plain, gemm_plain_f64, gemm_plain_c32, gemm_convert_f32,
// gemm_quantize_e4m3): the addresses in the loaded library
PyObject *fast_bind(PyObject *, PyObject *args) {
    unsigned long long a[5];
    if (!PyArg_ParseTuple(args, "KKKKK", &a[0], &a[1], &a[2], &a[3], &a[4])) return nullptr;
    g_plain = (PlainFn)a[0];
    g_f64 = (SameTypeF64Fn)a[1];
    g_c32 = (SameTypeC32Fn)a[2];
    g_convert = (ConvertFn)a[3];
    g_quantize = (QuantizeFn)a[4];
    Py_RETURN_NONE;
}

PyMethodDef kMethods[] = {
    {"gemm", (PyCFunction)(void (*)(void))fast_gemm, METH_FASTCALL, nullptr},
    {"gemm_same", (PyCFunction)(void (*)(void))fast_same, METH_FASTCALL, nullptr},
    {"convert", (PyCFunction)(void (*)(void))fast_convert, METH_FASTCALL, nullptr},
    {"quantize", (PyCFunction)(void (*)(void))fast_quantize, METH_FASTCALL, nullptr},
    {"bind", fast_bind, METH_VARARGS, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall(void) { return PyModule_Create(&kModule); }
