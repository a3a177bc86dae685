// Argument marshalling of the token-mixer calls for Python: checks the tensors, fills the
// descriptor and calls the C entry points of libjetvit.so.  What binding.py did through ctypes
// structures took 7 to 10 us of host time per call, as long as the kernels of a small problem
// (256 tokens x 6 heads: 13.2 us a call, host-bound, against 11 us of kernels); here it is below 1 us.
// Every function returns the entry point's status; binding.py turns it into an exception.  The
// interpreter lock is released around the entry points, as ctypes does, so that a launch that waits
// for room in the queue holds up no other thread.
#include <Python.h>

#include <ATen/hip/impl/HIPStreamMasqueradingAsCUDA.h>
#include <torch/csrc/autograd/python_variable.h>

#include "jetvit.h"

namespace {

const at::Tensor *tensor_arg(PyObject *obj) {
    if (!THPVariable_Check(obj)) {
        PyErr_SetString(PyExc_TypeError, "q, k, v, o must be torch tensors");
        return nullptr;
    }
    return &THPVariable_Unpack(obj);
}

bool dtype_code(const at::Tensor &t, jv_dtype *out) {
    if (t.scalar_type() == at::kFloat) *out = JV_F32;
    else if (t.scalar_type() == at::kBFloat16) *out = JV_BF16;
    else {
        PyErr_SetString(PyExc_TypeError, "unsupported dtype");
        return false;
    }
    return true;
}

bool pair_arg(PyObject *seq, int32_t *a, int32_t *b) {
    PyObject *fast = PySequence_Fast(seq, "expected a pair of integers");
    if (!fast) return false;
    bool ok = PySequence_Fast_GET_SIZE(fast) == 2;
    if (!ok) PyErr_SetString(PyExc_ValueError, "expected a pair of integers");
    if (ok) {
        const long x = PyLong_AsLong(PySequence_Fast_GET_ITEM(fast, 0)), y = PyLong_AsLong(PySequence_Fast_GET_ITEM(fast, 1));
        ok = !PyErr_Occurred();
        if (ok && (x != (int32_t)x || y != (int32_t)y)) {
            PyErr_SetString(PyExc_OverflowError, "grid or window side does not fit 32 bits");
            ok = false;
        }
        *a = (int32_t)x;
        *b = (int32_t)y;
    }
    Py_DECREF(fast);
    return ok;
}

struct Call {
    jv_attn_desc desc;
    const void *q, *k, *v;
    void *o, *stream;
};

bool stream_arg(PyObject *obj, void **stream) {
    if (obj == Py_None) {
        *stream = at::hip::getCurrentHIPStreamMasqueradingAsCUDA().stream();
        return true;
    }
    PyObject *raw = PyObject_GetAttrString(obj, "cuda_stream");
    if (!raw) return false;
    *stream = PyLong_AsVoidPtr(raw);
    Py_DECREF(raw);
    return !PyErr_Occurred();
}

// args: q, k, v, o, grid
bool mixer_args(PyObject *const *args, PyObject *stream, Call *c) {
    const at::Tensor *t[4];
    for (int i = 0; i < 4; ++i)
        if (!(t[i] = tensor_arg(args[i]))) return false;
    jv_attn_desc &d = c->desc;
    if (!pair_arg(args[4], &d.grid_h, &d.grid_w)) return false;
    if (t[0]->dim() != 4) {
        PyErr_SetString(PyExc_ValueError, "tensors must be [batch, heads, N, head_dim] views with a contiguous last axis");
        return false;
    }
    const auto shape = t[0]->sizes();
    if (shape[2] < (int64_t)d.grid_h * d.grid_w) {
        PyErr_SetString(PyExc_ValueError, "fewer tokens than grid cells");
        return false;
    }
    jv_strides *strides[4] = {&d.q, &d.k, &d.v, &d.o};
    for (int i = 0; i < 4; ++i) {
        if (t[i]->sizes() != shape) {
            PyErr_SetString(PyExc_ValueError, "q, k, v, o must share one shape");
            return false;
        }
        if (i < 3 && t[i]->scalar_type() != t[0]->scalar_type()) {
            PyErr_SetString(PyExc_TypeError, "q, k, v must share one dtype");
            return false;
        }
        if (!t[i]->is_cuda()) {
            PyErr_SetString(PyExc_ValueError, "tensors must live on the GPU");
            return false;
        }
        const auto s = t[i]->strides();
        if (s[3] != 1) {
            PyErr_SetString(PyExc_ValueError, "tensors must be [batch, heads, N, head_dim] views with a contiguous last axis");
            return false;
        }
        *strides[i] = {s[0], s[1], s[2]};
    }
    if (!dtype_code(*t[0], &d.dtype) || !dtype_code(*t[3], &d.o_dtype)) return false;
    for (int i : {0, 1, 3})
        if (shape[i] != (int32_t)shape[i]) {
            PyErr_SetString(PyExc_OverflowError, "tensor axis does not fit 32 bits");
            return false;
        }
    d.batch = (int32_t)shape[0];
    d.heads = (int32_t)shape[1];
    d.head_dim = (int32_t)shape[3];
    const int64_t prefix = shape[2] - (int64_t)d.grid_h * d.grid_w;
    d.n_prefix = prefix > 1 << 30 ? 1 << 30 : (int32_t)prefix;  // (the entry point refuses more than 64)
    c->q = t[0]->data_ptr();
    c->k = t[1]->data_ptr();
    c->v = t[2]->data_ptr();
    c->o = t[3]->data_ptr();
    return stream_arg(stream, &c->stream);
}

// f() without the interpreter lock.
template <typename F>
jv_status unlocked(F f) {
    jv_status st;
    Py_BEGIN_ALLOW_THREADS
    st = f();
    Py_END_ALLOW_THREADS
    return st;
}

bool arg_count(Py_ssize_t n, Py_ssize_t want) {
    if (n == want) return true;
    PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
    return false;
}

bool workspace_arg(PyObject *obj, void **ptr, size_t *bytes) {
    const at::Tensor *t = tensor_arg(obj);
    if (!t) return false;
    *ptr = t->data_ptr();
    *bytes = t->nbytes();
    return true;
}

// (q, k, v, o, grid, eps, workspace, stream)
PyObject *linear_attn_fwd(PyObject *, PyObject *const *a, Py_ssize_t n) {
    Call c;
    void *ws;
    size_t bytes;
    if (!arg_count(n, 8) || !mixer_args(a, a[7], &c)) return nullptr;
    const double eps = PyFloat_AsDouble(a[5]);
    if ((eps == -1.0 && PyErr_Occurred()) || !workspace_arg(a[6], &ws, &bytes)) return nullptr;
    return PyLong_FromLong(unlocked([&] { return jv_linear_attn_fwd(&c.desc, c.q, c.k, c.v, c.o, (float)eps, ws, bytes, c.stream); }));
}

// One fp32 device tensor of the convolution's parameters.
bool param_arg(PyObject *obj, const float **out, int64_t *rows) {
    const at::Tensor *t = tensor_arg(obj);
    if (!t) return false;
    if (t->scalar_type() != at::kFloat || !t->is_cuda() || !t->is_contiguous()) {
        PyErr_SetString(PyExc_ValueError, "convolution parameters must be contiguous fp32 device tensors");
        return false;
    }
    *out = (const float *)t->data_ptr();
    if (rows) *rows = t->dim() > 0 ? t->size(0) : 0;
    return true;
}

// static_kernel, squeeze, ksize, token as make_dwc_params of binding.py takes them
bool dwc_args(PyObject *kernel, PyObject *squeeze, PyObject *ksize, PyObject *token, jv_dwc_params *p) {
    *p = {JV_DWC_NONE, 3, 0, nullptr, nullptr, nullptr, nullptr, nullptr};
    if ((kernel != Py_None) + (squeeze != Py_None) + (token != Py_None) > 1) {
        PyErr_SetString(PyExc_ValueError, "give a static kernel or one set of generator weights, not several");
        return false;
    }
    const long k = PyLong_AsLong(ksize);
    if (k == -1 && PyErr_Occurred()) return false;
    p->ksize = k == (int32_t)k ? (int32_t)k : -1;
    if (kernel != Py_None) {
        p->mode = JV_DWC_STATIC;
        return param_arg(kernel, &p->static_kernel, nullptr);
    }
    PyObject *weights = squeeze != Py_None ? squeeze : token;
    if (weights == Py_None) return true;
    p->mode = squeeze != Py_None ? JV_DWC_SQUEEZE_DYNAMIC : JV_DWC_TOKEN_DYNAMIC;
    PyObject *fast = PySequence_Fast(weights, "generator weights must be (w1, b1, w2, b2)");
    if (!fast) return false;
    bool ok = PySequence_Fast_GET_SIZE(fast) == 4;
    if (!ok) PyErr_SetString(PyExc_ValueError, "generator weights must be (w1, b1, w2, b2)");
    const float **dst[4] = {&p->w1, &p->b1, &p->w2, &p->b2};
    int64_t hidden = 0;
    try {
        for (int i = 0; ok && i < 4; ++i) ok = param_arg(PySequence_Fast_GET_ITEM(fast, i), dst[i], i == 0 ? &hidden : nullptr);
    } catch (...) {
        Py_DECREF(fast);
        throw;
    }
    p->hidden = (int32_t)hidden;
    Py_DECREF(fast);
    return ok;
}

// (q, k, v, o, grid, eps, static_kernel, squeeze, ksize, token, focus_p, workspace, stream); focus_p 0: the ReLU map
PyObject *linear_block_fwd(PyObject *, PyObject *const *a, Py_ssize_t n) {
    Call c;
    jv_dwc_params dwc;
    void *ws;
    size_t bytes;
    if (!arg_count(n, 13) || !mixer_args(a, a[12], &c) || !dwc_args(a[6], a[7], a[8], a[9], &dwc)) return nullptr;
    const double eps = PyFloat_AsDouble(a[5]);
    if (eps == -1.0 && PyErr_Occurred()) return nullptr;
    const long focus = PyLong_AsLong(a[10]);
    if ((focus == -1 && PyErr_Occurred()) || !workspace_arg(a[11], &ws, &bytes)) return nullptr;
    return PyLong_FromLong(unlocked([&] {
        return focus == 0 ? jv_linear_block_fwd(&c.desc, c.q, c.k, c.v, c.o, (float)eps, &dwc, ws, bytes, c.stream)
                          : jv_linear_block_focused_fwd(&c.desc, c.q, c.k, c.v, c.o, (float)eps, (int32_t)focus, &dwc, ws, bytes, c.stream);
    }));
}

// (q, k, v, o, grid, window, scale, stream)
PyObject *window_attn_fwd(PyObject *, PyObject *const *a, Py_ssize_t n) {
    Call c;
    int32_t wh, ww;
    if (!arg_count(n, 8) || !mixer_args(a, a[7], &c) || !pair_arg(a[5], &wh, &ww)) return nullptr;
    const double scale = PyFloat_AsDouble(a[6]);
    if (scale == -1.0 && PyErr_Occurred()) return nullptr;
    return PyLong_FromLong(unlocked([&] { return jv_window_attn_fwd(&c.desc, c.q, c.k, c.v, c.o, wh, ww, (float)scale, c.stream); }));
}

// (q, k, v, o, grid, scale, stream)
PyObject *full_attn_fwd(PyObject *, PyObject *const *a, Py_ssize_t n) {
    Call c;
    if (!arg_count(n, 7) || !mixer_args(a, a[6], &c)) return nullptr;
    const double scale = PyFloat_AsDouble(a[5]);
    if (scale == -1.0 && PyErr_Occurred()) return nullptr;
    return PyLong_FromLong(unlocked([&] { return jv_full_attn_fwd(&c.desc, c.q, c.k, c.v, c.o, (float)scale, c.stream); }));
}

// Tensors without memory of their own (under tracing or vmap) throw where their pointer or strides
// are asked for: a Python exception, not the end of the process.
template <PyObject *(*F)(PyObject *, PyObject *const *, Py_ssize_t)>
PyObject *guarded(PyObject *self, PyObject *const *a, Py_ssize_t n) {
    try {
        return F(self, a, n);
    } catch (const c10::Error &e) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, e.what_without_backtrace());
    } catch (const std::exception &e) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, e.what());
    }
    return nullptr;
}

PyMethodDef methods[] = {
    {"linear_attn_fwd", (PyCFunction)(void *)guarded<linear_attn_fwd>, METH_FASTCALL, nullptr},
    {"linear_block_fwd", (PyCFunction)(void *)guarded<linear_block_fwd>, METH_FASTCALL, nullptr},
    {"window_attn_fwd", (PyCFunction)(void *)guarded<window_attn_fwd>, METH_FASTCALL, nullptr},
    {"full_attn_fwd", (PyCFunction)(void *)guarded<full_attn_fwd>, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&module); }
