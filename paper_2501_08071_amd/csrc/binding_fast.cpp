// The Python entry points' way to the C ABI for the usual call: torch tensors on the GPU, right shapes, right types.
//
// A small launch takes the GPU 3 to 6 us.  Looking at each tensor from Python (dtype, shape, contiguity, address), asking torch
// for the current stream and the ctypes call took 7.2 to 9.8 us (row softmax to product), so the host was what such a call waited
// for; from here it is 3.2 to 3.4, the launch itself most of it.  Every function takes the arguments of its namesake in binding.py and returns its result,
// or None for anything out of the ordinary -- whatever is not exactly a tensor with memory of its own on the GPU, a wrong shape
// or type, a status other than 0 (nothing has been launched then) -- and binding.py goes through its own checks, which say what
// is wrong.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <climits>

#include "../../include/attn.h"
#include "../../include/gemm.h"
#include "../../include/rowops.h"

namespace {

// the entry points of the library that binding.py has loaded
struct {
    decltype(&attn_fwd) attn;
    decltype(&attn_fwd_o16) attn_o16;
    decltype(&softmax_rows_fwd) softmax;
    decltype(&rmsnorm_fwd) rmsnorm;
    decltype(&gemm_leakyrelu_fwd) gemm;
} abi;

// A contiguous GPU tensor with memory of its own, or null.
const at::Tensor* gpu_tensor(PyObject* o) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    return t.defined() && t.has_storage() && t.is_cuda() && t.layout() == at::kStrided && t.is_contiguous() ? &t : nullptr;
}
int type_of(const at::Tensor& t) {
    const auto s = t.scalar_type();
    return s == at::kHalf ? 0 : s == at::kBFloat16 ? 1 : -1;
}
bool fits_int(int64_t n) { return n <= INT_MAX; }
// a plain number as Python's float() and int() would take it
bool real(PyObject* o, double& x) {
    if (!PyFloat_CheckExact(o) && !PyLong_CheckExact(o)) return false;
    x = PyFloat_AsDouble(o);
    return !(x == -1.0 && PyErr_Occurred());
}
bool flag(PyObject* o, int& x) {
    if (!PyBool_Check(o) && !PyLong_CheckExact(o)) return false;
    x = PyObject_IsTrue(o);
    return true;
}
// the stream handle: of the torch stream given, or of the current one on t's device
bool stream_of(PyObject* o, const at::Tensor& t, void*& st) {
    if (o == Py_None) {
        st = c10::hip::getCurrentHIPStream(t.device().index()).stream();
        return true;
    }
    PyObject* h = PyObject_GetAttrString(o, "cuda_stream");
    if (h == nullptr) return false;
    st = PyLong_AsVoidPtr(h);
    Py_DECREF(h);
    return !PyErr_Occurred();
}

// Launching and allocating may wait for the GPU, and what the GPU waits for may be Python's (a host function in a stream):
// both run without the interpreter's lock, as a call by way of ctypes does.
struct NoLock {
    PyThreadState* s = PyEval_SaveThread();
    ~NoLock() { PyEval_RestoreThread(s); }
};
at::Tensor new_tensor(at::IntArrayRef sizes, const at::TensorOptions& opt) {
    NoLock _;
    return at::empty(sizes, opt.requires_grad(false));
}

// What any of the functions below may throw (memory for an output, a device that is gone) is left to binding.py's own way.
template <class F>
PyObject* guarded(Py_ssize_t given, Py_ssize_t wanted, F f) {
    if (given != wanted) {
        PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
        return nullptr;
    }
    PyObject* r = nullptr;
    try {
        if (!at::impl::torch_function_mode_enabled()) r = f();
    } catch (...) {
        r = nullptr;
    }
    if (r != nullptr) return r;
    PyErr_Clear();
    Py_RETURN_NONE;
}

template <class F, class... T>
bool launched(F call, const T&... t) {
    return [&](auto... p) {
        NoLock _;
        return call(p...) == 0;
    }(t.mutable_data_ptr()...);
}

// (q, k, v, causal, scale, o, lse, stream, want_lse, o16) -> (o, lse)
PyObject* fast_attn(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 10, [&]() -> PyObject* {
        const at::Tensor *q = gpu_tensor(a[0]), *k = gpu_tensor(a[1]), *v = gpu_tensor(a[2]);
        if (!q || !k || !v) return nullptr;
        const int dt = type_of(*q);
        if (dt < 0 || type_of(*k) != dt || type_of(*v) != dt || q->dim() != 4 || k->sizes() != q->sizes() || v->sizes() != q->sizes()) return nullptr;
        const auto z = q->sizes();
        if (!fits_int(z[0]) || !fits_int(z[1]) || !fits_int(z[2]) || !fits_int(z[3])) return nullptr;
        int causal, want_lse, o16, rc;
        double scale;
        void* st;
        if (!flag(a[3], causal) || !real(a[4], scale) || !flag(a[8], want_lse) || !flag(a[9], o16) || !stream_of(a[7], *q, st)) return nullptr;
        const auto odt = o16 ? q->scalar_type() : at::kFloat;
        at::Tensor o_new, lse_new;
        const at::Tensor *o, *lse = nullptr;
        if (a[5] == Py_None) o = &(o_new = new_tensor(z, q->options().dtype(odt)));
        else if (!(o = gpu_tensor(a[5])) || o->scalar_type() != odt || o->sizes() != z) return nullptr;
        if (a[6] != Py_None) {
            if (!(lse = gpu_tensor(a[6])) || lse->scalar_type() != at::kFloat || lse->sizes() != z.slice(0, 3)) return nullptr;
        } else if (want_lse) {
            lse = &(lse_new = new_tensor(z.slice(0, 3), q->options().dtype(at::kFloat)));
        }
        float* l = lse ? (float*)lse->mutable_data_ptr() : nullptr;
        const int B = (int)z[0], H = (int)z[1], S = (int)z[2], D = (int)z[3];
        const void *qp = q->mutable_data_ptr(), *kp = k->mutable_data_ptr(), *vp = v->mutable_data_ptr();
        void* op = o->mutable_data_ptr();
        {
            NoLock _;
            rc = o16 ? abi.attn_o16(qp, kp, vp, op, l, B, H, S, D, causal, (float)scale, dt, st)
                     : abi.attn(qp, kp, vp, (float*)op, l, B, H, S, D, causal, (float)scale, dt, st);
        }
        if (rc != 0) return nullptr;
        PyObject* po = a[5] != Py_None ? Py_NewRef(a[5]) : THPVariable_Wrap(o_new);
        PyObject* pl = lse_new.defined() ? THPVariable_Wrap(lse_new) : Py_NewRef(a[6]);
        PyObject* r = po && pl ? PyTuple_Pack(2, po, pl) : nullptr;
        Py_XDECREF(po);
        Py_XDECREF(pl);
        return r;
    });
}

// x [..., d] and y of its shape and type (allocated if None); the rows
const at::Tensor* row_operands(PyObject* px, PyObject* py, at::Tensor& y_new, const at::Tensor*& y, long long& rows, int& d, int& dt) {
    const at::Tensor* x = gpu_tensor(px);
    if (!x || (dt = type_of(*x)) < 0 || x->dim() < 1) return nullptr;
    const int64_t n = x->sizes().back();
    if (!fits_int(n)) return nullptr;
    if (py == Py_None) y = &(y_new = new_tensor(x->sizes(), x->options()));
    else if (!(y = gpu_tensor(py)) || y->scalar_type() != x->scalar_type() || y->sizes() != x->sizes()) return nullptr;
    d = (int)n;
    rows = n ? x->numel() / n : 0;
    return x;
}
PyObject* given_or_new(PyObject* given, const at::Tensor& fresh) { return given != Py_None ? Py_NewRef(given) : THPVariable_Wrap(fresh); }

// (x, y, stream) -> y
PyObject* fast_softmax(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 3, [&]() -> PyObject* {
        at::Tensor y_new;
        const at::Tensor* y;
        long long rows;
        int d, dt;
        void* st;
        const at::Tensor* x = row_operands(a[0], a[1], y_new, y, rows, d, dt);
        if (!x || !stream_of(a[2], *x, st)) return nullptr;
        if (launched([&](void* xp, void* yp) { return abi.softmax(xp, yp, rows, d, dt, st); }, *x, *y)) return given_or_new(a[1], y_new);
        return nullptr;
    });
}

// (x, w, eps, y, stream) -> y
PyObject* fast_rmsnorm(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 5, [&]() -> PyObject* {
        at::Tensor y_new;
        const at::Tensor* y;
        long long rows;
        int d, dt;
        void* st;
        double eps;
        const at::Tensor *x = row_operands(a[0], a[3], y_new, y, rows, d, dt), *w = gpu_tensor(a[1]);
        if (!x || !w || w->scalar_type() != x->scalar_type() || w->dim() != 1 || w->sizes()[0] != d) return nullptr;
        if (!real(a[2], eps) || !stream_of(a[4], *x, st)) return nullptr;
        if (launched([&](void* xp, void* wp, void* yp) { return abi.rmsnorm(xp, wp, yp, rows, d, (float)eps, dt, st); }, *x, *w, *y))
            return given_or_new(a[3], y_new);
        return nullptr;
    });
}

// (a, b, slope, c, stream) -> c
PyObject* fast_gemm(PyObject*, PyObject* const* g, Py_ssize_t n) {
    return guarded(n, 5, [&]() -> PyObject* {
        const at::Tensor *a = gpu_tensor(g[0]), *b = gpu_tensor(g[1]), *c;
        if (!a || !b) return nullptr;
        const int dt = type_of(*a);
        const int64_t dim = a->dim();
        if (dt < 0 || type_of(*b) != dt || b->dim() != dim || (dim != 2 && dim != 3)) return nullptr;
        const int64_t batch = dim == 3 ? a->size(0) : 1, M = a->size(dim - 2), K = a->size(dim - 1), N = b->size(dim - 1);
        if ((dim == 3 && b->size(0) != batch) || b->size(dim - 2) != K) return nullptr;
        if (!fits_int(batch) || !fits_int(M) || !fits_int(K) || !fits_int(N)) return nullptr;
        double slope;
        void* st;
        if (!real(g[2], slope) || !stream_of(g[4], *a, st)) return nullptr;
        const int64_t shape3[3] = {batch, M, N};
        const at::IntArrayRef shape(shape3 + (3 - dim), dim);
        at::Tensor c_new;
        if (g[3] == Py_None) c = &(c_new = new_tensor(shape, a->options()));
        else if (!(c = gpu_tensor(g[3])) || c->scalar_type() != a->scalar_type() || c->sizes() != shape) return nullptr;
        if (launched([&](void* ap, void* bp, void* cp) { return abi.gemm(ap, bp, cp, (int)batch, (int)M, (int)N, (int)K, (float)slope, dt, st); }, *a, *b, *c))
            return given_or_new(g[3], c_new);
        return nullptr;
    });
}

// the addresses of the library's entry points, in the order of `abi`
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 5) {
        PyErr_SetString(PyExc_TypeError, "five addresses");
        return nullptr;
    }
    void* p[5];
    for (int i = 0; i < 5; ++i) p[i] = PyLong_AsVoidPtr(a[i]);
    if (PyErr_Occurred()) return nullptr;
    abi = {reinterpret_cast<decltype(abi.attn)>(p[0]), reinterpret_cast<decltype(abi.attn_o16)>(p[1]), reinterpret_cast<decltype(abi.softmax)>(p[2]),
           reinterpret_cast<decltype(abi.rmsnorm)>(p[3]), reinterpret_cast<decltype(abi.gemm)>(p[4])};
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"bind", (PyCFunction)(void*)bind, METH_FASTCALL, nullptr},
                         {"attn_fwd", (PyCFunction)(void*)fast_attn, METH_FASTCALL, nullptr},
                         {"softmax_rows_fwd", (PyCFunction)(void*)fast_softmax, METH_FASTCALL, nullptr},
                         {"rmsnorm_fwd", (PyCFunction)(void*)fast_rmsnorm, METH_FASTCALL, nullptr},
                         {"gemm_leakyrelu_fwd", (PyCFunction)(void*)fast_gemm, METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding_fast", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding_fast(void) { return PyModule_Create(&module); }
