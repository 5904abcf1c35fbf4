// The binding's calls on torch tensors, for the plain case: operands that are ordinary dense
// tensors on the matrix's GPU with the shapes, strides and formats the library takes.  The checks are
// those of binding.py, made natively because a launch takes the host less time than they take in
// Python (a 256 x 256 by 256 x 64 product: 8.4 us per call from Python, 3.5 us from here, of which the HIP launch is 3).  Whatever is not
// the plain case - wrong shapes, host tensors, subclasses, tensors inside a transform - returns None,
// and binding.py goes through its own checks, which raise or take the general way.
//
// No state is kept between calls but the plan, which its Matrix owns: the handle, what
// shflbw_info says about it and the GPU it is bound to.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <c10/core/impl/VirtualGuardImpl.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

#include "shflbw.h"

namespace {

typedef decltype(&shflbw_spmm) spmm_fn;
typedef decltype(&shflbw_conv2d) conv2d_fn;
typedef decltype(&shflbw_layernorm_transpose) layernorm_fn;

spmm_fn g_spmm = nullptr;            // the entry points of the library that binding.py has loaded
conv2d_fn g_conv2d = nullptr;
layernorm_fn g_layernorm = nullptr;
PyObject* g_raw_stream = nullptr;    // device index -> current stream's handle

struct Plan {
    shflbw_matrix* A;
    int64_t M, K;
    c10::ScalarType dtype;
    int device;
};
const char* const PLAN = "shflbw plan";

// an ordinary dense tensor on GPU `device` that no transform, mode or lazy view stands behind
bool plain(PyObject* o, int device, const at::Tensor*& t)
{
    if (!THPVariable_CheckExact(o)) return false;
    t = &THPVariable_Unpack(o);
    if (!t->defined()) return false;
    const c10::DispatchKeySet known({c10::DispatchKey::CUDA, c10::DispatchKey::ADInplaceOrView, c10::DispatchKey::AutogradCUDA,
                                     c10::DispatchKey::AutocastCUDA});
    const c10::TensorImpl* impl = t->unsafeGetTensorImpl();
    return (impl->key_set() - known).highestFunctionalityKey() == c10::DispatchKey::Undefined && t->is_cuda() && t->layout() == at::kStrided && t->has_storage() &&
           t->device().index() == device;
}

// -1: not an output format
int ydtype_of(c10::ScalarType s)
{
    return s == at::kHalf ? SHFLBW_F16 : s == at::kBFloat16 ? SHFLBW_BF16 : s == at::kFloat ? SHFLBW_F32 : -1;
}

int current_device() { return c10::impl::VirtualGuardImpl(c10::DeviceType::CUDA).getDevice().index(); }

// the current device's current stream; false with a Python error set
bool current_stream(void*& stream)
{
    PyObject* index = PyLong_FromLong(current_device());
    if (!index) return false;
    PyObject* raw = PyObject_CallOneArg(g_raw_stream, index);
    Py_DECREF(index);
    if (!raw) return false;
    stream = PyLong_AsVoidPtr(raw);
    Py_DECREF(raw);
    return !PyErr_Occurred();
}

bool small_int(PyObject* o, int& v)
{
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    const long x = PyLong_AsLongAndOverflow(o, &overflow);
    if (overflow || x < INT32_MIN || x > INT32_MAX) return false;
    v = (int)x;
    return true;
}
bool int_pair(PyObject* o, int& a, int& b)
{
    return PyTuple_CheckExact(o) && PyTuple_GET_SIZE(o) == 2 && small_int(PyTuple_GET_ITEM(o, 0), a) &&
           small_int(PyTuple_GET_ITEM(o, 1), b);
}

// Releases the interpreter lock for as long as it lives, and holds it again when an exception passes by.
struct Unlocked {
    PyThreadState* state = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(state); }
};
template <class F>
int unlocked(F&& f)
{
    Unlocked u;
    return f();
}

template <class F>
PyObject* guarded(F&& f)
{
    try {
        return f();
    } catch (...) {          // a C++ exception of torch's: binding.py meets the same tensor and reports it
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

// spmm(plan, X, Y) -> status, or None
PyObject* spmm(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    if (n != 3) { PyErr_SetString(PyExc_TypeError, "spmm(plan, X, Y)"); return nullptr; }
    const Plan* p = static_cast<const Plan*>(PyCapsule_GetPointer(args[0], PLAN));
    if (!p) return nullptr;
    return guarded([&]() -> PyObject* {
        const at::Tensor *X, *Y;
        if (!plain(args[1], p->device, X) || !plain(args[2], p->device, Y)) Py_RETURN_NONE;
        const int yd = ydtype_of(Y->scalar_type());
        if (X->scalar_type() != p->dtype || X->dim() != 2 || Y->dim() != 2 || yd < 0) Py_RETURN_NONE;
        const int64_t N = X->size(1);
        if (X->size(0) != p->K || Y->size(0) != p->M || Y->size(1) != N || N < 1) Py_RETURN_NONE;
        if (N > 1 && (X->stride(1) != 1 || Y->stride(1) != 1)) Py_RETURN_NONE;
        if ((p->K > 1 && X->stride(0) < N) || (p->M > 1 && Y->stride(0) < N)) Py_RETURN_NONE;
        const int64_t ldx = p->K > 1 ? X->stride(0) : N, ldy = p->M > 1 ? Y->stride(0) : N;
        const void* x = X->const_data_ptr();
        void* y = Y->data_ptr();
        void* stream;
        if (!current_stream(stream)) return nullptr;
        return PyLong_FromLong(unlocked([&] {
            return g_spmm(p->A, x, ldx, y, ldy, N, (shflbw_dtype)yd, stream);
        }));
    });
}

// conv2d(plan, inp, R, S, stride, pad, chwn, out) -> status, or None
PyObject* conv2d(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    if (n != 8) { PyErr_SetString(PyExc_TypeError, "conv2d(plan, inp, R, S, stride, pad, chwn, out)"); return nullptr; }
    const Plan* p = static_cast<const Plan*>(PyCapsule_GetPointer(args[0], PLAN));
    if (!p) return nullptr;
    return guarded([&]() -> PyObject* {
        const at::Tensor *in, *out;
        int R, S, sh, sw, ph, pw;
        if (!plain(args[1], p->device, in) || !plain(args[7], p->device, out)) Py_RETURN_NONE;
        if (!small_int(args[2], R) || !small_int(args[3], S) || !int_pair(args[4], sh, sw) || !int_pair(args[5], ph, pw))
            Py_RETURN_NONE;
        const bool chwn = args[6] == Py_True;
        const int yd = ydtype_of(out->scalar_type());
        if (in->scalar_type() != p->dtype || in->dim() != 4 || out->dim() != 4 || yd < 0 || !in->is_contiguous() ||
            !out->is_contiguous())
            Py_RETURN_NONE;
        const int64_t B = in->size(chwn ? 3 : 0), C = in->size(chwn ? 0 : 1), H = in->size(chwn ? 1 : 2), W = in->size(chwn ? 2 : 3);
        const int64_t big = 1 << 20;
        if (B < 1 || B >= (1LL << 31) || C >= (1LL << 31) || H >= big || W >= big || R < 1 || S < 1 || R >= big || S >= big ||
            sh < 1 || sw < 1 || ph < 0 || pw < 0 || ph >= big || pw >= big)
            Py_RETURN_NONE;
        if ((int64_t)R * S > p->K || C * R * S != p->K || H + 2 * ph < R || W + 2 * pw < S) Py_RETURN_NONE;
        const int64_t Ho = (H + 2 * ph - R) / sh + 1, Wo = (W + 2 * pw - S) / sw + 1;
        if (out->size(chwn ? 3 : 0) != B || out->size(chwn ? 0 : 1) != p->M || out->size(chwn ? 1 : 2) != Ho ||
            out->size(chwn ? 2 : 3) != Wo)
            Py_RETURN_NONE;
        const void* x = in->const_data_ptr();
        void* y = out->data_ptr();
        void* stream;
        if (!current_stream(stream)) return nullptr;
        return PyLong_FromLong(unlocked([&] {
            return g_conv2d(p->A, x, y, (int)B, (int)C, (int)H, (int)W, R, S, sh, sw, ph, pw, chwn ? SHFLBW_CHWN : SHFLBW_NCHW,
                            (shflbw_dtype)yd, stream);
        }));
    });
}

// layernorm_transpose(x, gamma, beta, eps, normalize, out) -> status, or None
PyObject* layernorm_transpose(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    if (n != 6) { PyErr_SetString(PyExc_TypeError, "layernorm_transpose(x, gamma, beta, eps, normalize, out)"); return nullptr; }
    return guarded([&]() -> PyObject* {
        const at::Tensor *x, *out, *par[2] = {nullptr, nullptr};
        if (!THPVariable_CheckExact(args[0])) Py_RETURN_NONE;
        const int device = THPVariable_Unpack(args[0]).device().index();
        if (!plain(args[0], device, x) || !plain(args[5], device, out)) Py_RETURN_NONE;
        const c10::ScalarType dt = x->scalar_type();
        if ((dt != at::kHalf && dt != at::kBFloat16) || out->scalar_type() != dt || x->dim() != 2 || out->dim() != 2) Py_RETURN_NONE;
        const int64_t N = x->size(0), K = x->size(1);
        if (N < 1 || K < 1 || K > INT32_MAX || out->size(0) != K || out->size(1) != N || x->stride(1) != 1 || out->stride(1) != 1)
            Py_RETURN_NONE;
        if ((N > 1 && x->stride(0) < K) || (K > 1 && out->stride(0) < N)) Py_RETURN_NONE;
        for (int i = 0; i < 2; ++i) {
            if (args[1 + i] == Py_None) continue;
            if (!plain(args[1 + i], device, par[i])) Py_RETURN_NONE;
            if (par[i]->scalar_type() != dt || par[i]->dim() != 1 || par[i]->size(0) != K || !par[i]->is_contiguous()) Py_RETURN_NONE;
        }
        if (!PyFloat_CheckExact(args[3]) || !PyBool_Check(args[4])) Py_RETURN_NONE;
        const float eps = (float)PyFloat_AS_DOUBLE(args[3]);
        const int normalize = args[4] == Py_True;
        const void *xp = x->const_data_ptr(), *g = par[0] ? par[0]->const_data_ptr() : nullptr,
                   *b = par[1] ? par[1]->const_data_ptr() : nullptr;
        void* y = out->data_ptr();
        const int64_t ldx = N > 1 ? x->stride(0) : K, ldo = K > 1 ? out->stride(0) : N;
        void* stream;
        if (!current_stream(stream)) return nullptr;
        return PyLong_FromLong(unlocked([&] {
            return g_layernorm(xp, ldx, g, b, eps, normalize, y, ldo, N, (int)K, dt == at::kBFloat16 ? SHFLBW_BF16 : SHFLBW_F16, stream);
        }));
    });
}

// plan(handle, M, K, bf16, device index) -> capsule
PyObject* plan(PyObject*, PyObject* args)
{
    unsigned long long handle;
    long long M, K;
    int bf16, device;
    if (!PyArg_ParseTuple(args, "KLLpi", &handle, &M, &K, &bf16, &device)) return nullptr;
    Plan* p = new (std::nothrow) Plan{reinterpret_cast<shflbw_matrix*>((uintptr_t)handle), (int64_t)M, (int64_t)K,
                                      bf16 ? at::kBFloat16 : at::kHalf, device};
    if (!p) return PyErr_NoMemory();
    PyObject* c = PyCapsule_New(p, PLAN, [](PyObject* o) { delete static_cast<Plan*>(PyCapsule_GetPointer(o, PLAN)); });
    if (!c) delete p;
    return c;
}

// connect(address of shflbw_spmm, of shflbw_conv2d, of shflbw_layernorm_transpose, raw_stream)
PyObject* connect(PyObject*, PyObject* args)
{
    unsigned long long s, c, l;
    PyObject* raw;
    if (!PyArg_ParseTuple(args, "KKKO", &s, &c, &l, &raw)) return nullptr;
    g_spmm = reinterpret_cast<spmm_fn>((uintptr_t)s);
    g_conv2d = reinterpret_cast<conv2d_fn>((uintptr_t)c);
    g_layernorm = reinterpret_cast<layernorm_fn>((uintptr_t)l);
    Py_INCREF(raw);
    Py_XDECREF(g_raw_stream);
    g_raw_stream = raw;
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"connect", connect, METH_VARARGS, "Entry points of the loaded library and torch's raw-stream function."},
    {"plan", plan, METH_VARARGS, "What a call needs to know of one bound matrix."},
    {"spmm", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(&spmm)), METH_FASTCALL, "shflbw_spmm on plain tensors."},
    {"conv2d", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(&conv2d)), METH_FASTCALL, "shflbw_conv2d on plain tensors."},
    {"layernorm_transpose", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(&layernorm_transpose)), METH_FASTCALL,
     "shflbw_layernorm_transpose on plain tensors."},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_torch_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// The caller compares TORCH_VERSION with the torch it runs on before any call: tensors are read in its own layout.
PyMODINIT_FUNC PyInit__torch_calls(void)
{
    PyObject* m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "TORCH_VERSION", SHFLBW_TORCH_VERSION) < 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
