// The forward calls of binding.py for the ordinary case, in native code: plain contiguous fp32 tensors on the current device, the
// output given, the current stream.  Anything else is declined (None) and takes the Python lines, which also raise the errors.
//
// A small layer's call is bound by the host (kernels of 3-5 us): of 5.1 us from Python 3.1 were the library's call, 2.4 of them the
// launch, and the rest Python's look at two tensors, some twelve attribute and method calls.  Read from the tensors' own fields they
// cost 0.2 us.
#include <Python.h>

#include <torch/csrc/autograd/python_variable.h>

namespace {

using ForwardFn = int (*)(void *, const float *, float *, int32_t, void *);
using FusedFn = int (*)(void *, const float *, float *, int32_t, const float *, int32_t, void *);

// A handle, the library's calls that take it and the shapes it was created for.
struct Layer {
    void *handle;
    ForwardFn forward, noalloc;
    FusedFn fused, fc;
    PyObject *current_device;   // () -> index
    PyObject *current_stream;   // index -> raw handle
    int64_t in[3], out[3];
};
const char kLayer[] = "sconv layer";

// The tensor, if it is a plain one the kernels can read: fp32, contiguous, on a GPU, with memory of its own.
const at::Tensor *plain(PyObject *o)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || t.layout() != at::kStrided || !t.is_cuda() || t.scalar_type() != at::kFloat || !t.has_storage() || !t.is_contiguous()) return nullptr;
    return &t;
}

bool shaped(const at::Tensor &t, std::initializer_list<int64_t> dims) { return t.sizes() == at::IntArrayRef(dims.begin(), dims.size()); }

// The current stream of x's device as an integer object's value; false if that device is not the current one.
bool stream_of(const Layer &l, const at::Tensor &x, void **stream)
{
    const int64_t index = x.get_device();
    PyObject *d = PyObject_CallNoArgs(l.current_device);
    const long current = d ? PyLong_AsLong(d) : -1;
    Py_XDECREF(d);
    if (current != index) return false;
    PyObject *i = PyLong_FromLong(current), *s = i ? PyObject_CallOneArg(l.current_stream, i) : nullptr;
    Py_XDECREF(i);
    if (!s) return false;
    *stream = PyLong_AsVoidPtr(s);
    Py_DECREF(s);
    return !PyErr_Occurred();
}

PyObject *declined()
{
    PyErr_Clear();
    Py_RETURN_NONE;
}

enum Entry { kForward, kNoalloc, kFused, kFc };

PyObject *run(Entry entry, PyObject *layer, PyObject *x_, PyObject *bias_, PyObject *relu, PyObject *out_)
{
    if (layer == Py_None || out_ == Py_None) Py_RETURN_NONE;
    try {
        auto *l = static_cast<Layer *>(PyCapsule_GetPointer(layer, kLayer));
        const at::Tensor *x = l ? plain(x_) : nullptr, *out = x ? plain(out_) : nullptr, *bias = nullptr;
        if (!out) return declined();
        int64_t n;
        if (entry == kFc) {
            if (x->dim() != 2) return declined();
            n = x->size(1);
            if (!shaped(*x, {l->in[0], n}) || !shaped(*out, {l->out[0], n})) return declined();
        } else {
            if (x->dim() != 4) return declined();
            n = x->size(0);
            if (!shaped(*x, {n, l->in[0], l->in[1], l->in[2]}) || !shaped(*out, {n, l->out[0], l->out[1], l->out[2]})) return declined();
        }
        if (bias_ && bias_ != Py_None && (!(bias = plain(bias_)) || !shaped(*bias, {l->out[0]}))) return declined();
        const int on = relu ? PyObject_IsTrue(relu) : 0;
        const Layer c = *l;   // (another thread may destroy the handle's object meanwhile)
        void *stream;
        if (on < 0 || n > INT32_MAX || !stream_of(*l, *x, &stream)) return declined();
        const float *in = static_cast<const float *>(x->data_ptr()), *b = bias ? static_cast<const float *>(bias->data_ptr()) : nullptr;
        float *to = static_cast<float *>(out->data_ptr());
        int rc;
        Py_BEGIN_ALLOW_THREADS
        if (entry == kFused || entry == kFc) rc = (entry == kFc ? c.fc : c.fused)(c.handle, in, to, (int32_t)n, b, on, stream);
        else rc = (entry == kNoalloc ? c.noalloc : c.forward)(c.handle, in, to, (int32_t)n, stream);
        Py_END_ALLOW_THREADS
        return PyLong_FromLong(rc);
    } catch (...) {   // a tensor whose data cannot be had: the Python lines say so
        return declined();
    }
}

#define SCONV_ARGS(N) \
    if (n != N) { \
        PyErr_SetString(PyExc_TypeError, "wrong number of arguments"); \
        return nullptr; \
    }
PyObject *forward(PyObject *, PyObject *const *a, Py_ssize_t n) { SCONV_ARGS(3) return run(kForward, a[0], a[1], nullptr, nullptr, a[2]); }
PyObject *noalloc(PyObject *, PyObject *const *a, Py_ssize_t n) { SCONV_ARGS(3) return run(kNoalloc, a[0], a[1], nullptr, nullptr, a[2]); }
PyObject *fused(PyObject *, PyObject *const *a, Py_ssize_t n) { SCONV_ARGS(5) return run(kFused, a[0], a[1], a[2], a[3], a[4]); }
PyObject *fc(PyObject *, PyObject *const *a, Py_ssize_t n) { SCONV_ARGS(5) return run(kFc, a[0], a[1], a[2], a[3], a[4]); }

// layer(handle, forward, noalloc, fused, fc: addresses, current device, current stream: callables, C, H, W, K, OH, OW)
PyObject *layer(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    SCONV_ARGS(13)
    auto *l = new Layer;
    l->handle = PyLong_AsVoidPtr(a[0]);
    l->forward = (ForwardFn)PyLong_AsVoidPtr(a[1]);
    l->noalloc = (ForwardFn)PyLong_AsVoidPtr(a[2]);
    l->fused = (FusedFn)PyLong_AsVoidPtr(a[3]);
    l->fc = (FusedFn)PyLong_AsVoidPtr(a[4]);
    for (int i = 0; i < 3; ++i) {
        l->in[i] = PyLong_AsLongLong(a[7 + i]);
        l->out[i] = PyLong_AsLongLong(a[10 + i]);
    }
    PyObject *c = PyErr_Occurred() ? nullptr : PyCapsule_New(l, kLayer, [](PyObject *o) {
        auto *l = static_cast<Layer *>(PyCapsule_GetPointer(o, kLayer));
        Py_DECREF(l->current_device);
        Py_DECREF(l->current_stream);
        delete l;
    });
    if (!c) {
        delete l;
        return nullptr;
    }
    Py_INCREF(l->current_device = a[5]);
    Py_INCREF(l->current_stream = a[6]);
    return c;
}

#define SCONV_METHOD(F) {#F, (PyCFunction)(void (*)(void))F, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {SCONV_METHOD(layer), SCONV_METHOD(forward), SCONV_METHOD(noalloc), SCONV_METHOD(fused), SCONV_METHOD(fc),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_sconv_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

} // namespace

PyMODINIT_FUNC PyInit__sconv_call()
{
    PyObject *m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "torch_version", SCONV_TORCH_VERSION)) Py_CLEAR(m);
    return m;
}
