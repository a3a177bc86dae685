// Argument marshalling of the token-mixer calls for Python: checks the tensors, fills the
// descriptor and calls the C entry points of libjetvit.so.  Host time of a call, launches included,
// through ctypes structures / here: window or full attention 10.3 / 3.9 us, linear attention
// 13.7 / 7.4 us, the block with generated filters 25.4 / 20.3 us, where the kernels of a small problem take about 10.
// Only the ordinary forms are marshalled here: torch tensors with memory, pairs as tuples or lists.
// Every function returns the entry point's status, or None for arguments of any other form, valid
// or not, which binding.py then takes through ctypes: what is accepted, and the exceptions of what
// is not, are those of that path.  The interpreter lock is released around the entry points, as
// ctypes does, so that a launch that waits for room in the queue holds up no other thread.
#include <Python.h>

#include <ATen/hip/impl/HIPStreamMasqueradingAsCUDA.h>
#include <torch/csrc/autograd/python_variable.h>

#include "jetvit.h"

namespace {

// The readers below return false (or null) for a form that is left to binding.py; a Python error
// they leave set is cleared by `guarded`.
const at::Tensor *tensor_arg(PyObject *obj) { return THPVariable_Check(obj) ? &THPVariable_Unpack(obj) : nullptr; }

bool dtype_code(const at::Tensor &t, jv_dtype *out) {
    if (t.scalar_type() == at::kFloat) *out = JV_F32;
    else if (t.scalar_type() == at::kBFloat16) *out = JV_BF16;
    else return false;
    return true;
}

bool int_arg(PyObject *obj, int32_t *out) {
    const long x = PyLong_AsLong(obj);
    *out = (int32_t)x;
    return x == *out && !(x == -1 && PyErr_Occurred());
}

bool float_arg(PyObject *obj, float *out) {
    const double x = PyFloat_AsDouble(obj);
    *out = (float)x;
    return !(x == -1.0 && PyErr_Occurred());
}

// Items of a tuple or list of exactly n (borrowed references), or null.
PyObject **items_arg(PyObject *seq, Py_ssize_t n) {
    if (!PyTuple_Check(seq) && !PyList_Check(seq)) return nullptr;
    return PySequence_Fast_GET_SIZE(seq) == n ? PySequence_Fast_ITEMS(seq) : nullptr;
}

bool pair_arg(PyObject *seq, int32_t *a, int32_t *b) {
    PyObject **items = items_arg(seq, 2);
    return items && int_arg(items[0], a) && int_arg(items[1], b);
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
    if (!pair_arg(args[4], &d.grid_h, &d.grid_w) || t[0]->dim() != 4) return false;
    const auto shape = t[0]->sizes();
    const int64_t prefix = shape[2] - (int64_t)d.grid_h * d.grid_w;
    if (prefix < 0 || prefix != (int32_t)prefix) return false;
    jv_strides *strides[4] = {&d.q, &d.k, &d.v, &d.o};
    for (int i = 0; i < 4; ++i) {
        if (t[i]->sizes() != shape || !t[i]->is_cuda() || (i < 3 && t[i]->scalar_type() != t[0]->scalar_type())) return false;
        const auto s = t[i]->strides();
        if (s[3] != 1) return false;
        *strides[i] = {s[0], s[1], s[2]};
    }
    if (!dtype_code(*t[0], &d.dtype) || !dtype_code(*t[3], &d.o_dtype)) return false;
    for (int i : {0, 1, 3})
        if (shape[i] != (int32_t)shape[i]) return false;
    d.batch = (int32_t)shape[0];
    d.heads = (int32_t)shape[1];
    d.head_dim = (int32_t)shape[3];
    d.n_prefix = (int32_t)prefix;
    c->q = t[0]->data_ptr();
    c->k = t[1]->data_ptr();
    c->v = t[2]->data_ptr();
    c->o = t[3]->data_ptr();
    return stream_arg(stream, &c->stream);
}

// f() without the interpreter lock.
template <typename F>
PyObject *status_of(F f) {
    jv_status st;
    Py_BEGIN_ALLOW_THREADS
    st = f();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
}

bool workspace_arg(PyObject *obj, void **ptr, size_t *bytes) {
    const at::Tensor *t = tensor_arg(obj);
    if (!t) return false;
    *ptr = t->data_ptr();
    *bytes = t->nbytes();
    return true;
}

// (q, k, v, o, grid, eps, workspace, stream)
PyObject *linear_attn_fwd(PyObject *const *a) {
    Call c;
    float eps;
    void *ws;
    size_t bytes;
    if (!mixer_args(a, a[7], &c) || !float_arg(a[5], &eps) || !workspace_arg(a[6], &ws, &bytes)) return nullptr;
    return status_of([&] { return jv_linear_attn_fwd(&c.desc, c.q, c.k, c.v, c.o, eps, ws, bytes, c.stream); });
}

// One fp32 device tensor of the convolution's parameters; rows: the length of its first axis, if asked for.
bool param_arg(PyObject *obj, const float **out, int32_t *rows = nullptr) {
    const at::Tensor *t = tensor_arg(obj);
    if (!t || t->scalar_type() != at::kFloat || !t->is_cuda() || !t->is_contiguous()) return false;
    *out = (const float *)t->data_ptr();
    if (!rows) return true;
    if (t->dim() == 0 || t->size(0) != (int32_t)t->size(0)) return false;
    *rows = (int32_t)t->size(0);
    return true;
}

// static_kernel, squeeze, ksize, token as make_dwc_params of binding.py takes them
bool dwc_args(PyObject *kernel, PyObject *squeeze, PyObject *ksize, PyObject *token, jv_dwc_params *p) {
    *p = {JV_DWC_NONE, 3, 0, nullptr, nullptr, nullptr, nullptr, nullptr};
    if ((kernel != Py_None) + (squeeze != Py_None) + (token != Py_None) > 1 || !int_arg(ksize, &p->ksize)) return false;
    if (kernel != Py_None) {
        p->mode = JV_DWC_STATIC;
        return param_arg(kernel, &p->static_kernel);
    }
    PyObject *weights = squeeze != Py_None ? squeeze : token;
    if (weights == Py_None) return true;
    p->mode = squeeze != Py_None ? JV_DWC_SQUEEZE_DYNAMIC : JV_DWC_TOKEN_DYNAMIC;
    PyObject **w = items_arg(weights, 4);
    return w && param_arg(w[0], &p->w1, &p->hidden) && param_arg(w[1], &p->b1) && param_arg(w[2], &p->w2) && param_arg(w[3], &p->b2);
}

// (q, k, v, o, grid, eps, static_kernel, squeeze, ksize, token, focus_p, workspace, stream); focus_p 0: the ReLU map
PyObject *linear_block_fwd(PyObject *const *a) {
    Call c;
    jv_dwc_params dwc;
    float eps;
    int32_t focus;
    void *ws;
    size_t bytes;
    if (!mixer_args(a, a[12], &c) || !dwc_args(a[6], a[7], a[8], a[9], &dwc) || !float_arg(a[5], &eps) ||
        !int_arg(a[10], &focus) || !workspace_arg(a[11], &ws, &bytes))
        return nullptr;
    return status_of([&] {
        return focus == 0 ? jv_linear_block_fwd(&c.desc, c.q, c.k, c.v, c.o, eps, &dwc, ws, bytes, c.stream)
                          : jv_linear_block_focused_fwd(&c.desc, c.q, c.k, c.v, c.o, eps, focus, &dwc, ws, bytes, c.stream);
    });
}

// (q, k, v, o, grid, window, scale, stream)
PyObject *window_attn_fwd(PyObject *const *a) {
    Call c;
    int32_t wh, ww;
    float scale;
    if (!mixer_args(a, a[7], &c) || !pair_arg(a[5], &wh, &ww) || !float_arg(a[6], &scale)) return nullptr;
    return status_of([&] { return jv_window_attn_fwd(&c.desc, c.q, c.k, c.v, c.o, wh, ww, scale, c.stream); });
}

// (q, k, v, o, grid, scale, stream)
PyObject *full_attn_fwd(PyObject *const *a) {
    Call c;
    float scale;
    if (!mixer_args(a, a[6], &c) || !float_arg(a[5], &scale)) return nullptr;
    return status_of([&] { return jv_full_attn_fwd(&c.desc, c.q, c.k, c.v, c.o, scale, c.stream); });
}

// Tensors without memory of their own (under tracing or vmap) throw where their pointer or strides
// are asked for, and torch where it has no device for the current stream: left to binding.py too.
// Nothing throws behind an entry point, so no call is made twice.
template <PyObject *(*F)(PyObject *const *), Py_ssize_t ARGS>
PyObject *guarded(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (n != ARGS) {
        PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
        return nullptr;
    }
    try {
        if (PyObject *status = F(a)) return status;
    } catch (const std::exception &) {
    }
    PyErr_Clear();
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"linear_attn_fwd", (PyCFunction)(void *)guarded<linear_attn_fwd, 8>, METH_FASTCALL, nullptr},
    {"linear_block_fwd", (PyCFunction)(void *)guarded<linear_block_fwd, 13>, METH_FASTCALL, nullptr},
    {"window_attn_fwd", (PyCFunction)(void *)guarded<window_attn_fwd, 8>, METH_FASTCALL, nullptr},
    {"full_attn_fwd", (PyCFunction)(void *)guarded<full_attn_fwd, 7>, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&module); }
