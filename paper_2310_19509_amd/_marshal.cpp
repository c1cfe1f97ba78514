// The run calls' argument marshalling for the ordinary case: plain contiguous float32 tensors on a GPU, sizes as Python
// integers, the current stream.  One layer of a network on one image takes the GPU 3 to 5 us; the same checks and
// conversions through Python attributes and ctypes take the host 7.7 us a call, this takes 3.4 (3 of them the launch).
// Anything else (addresses, other streams, subclasses, wrapped tensors, errors) is answered with None, and the Python code of
// api.py, which has the checks and their messages, does it.
#include <Python.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <climits>

namespace {

typedef int (*LayerFn)(const void*, const float*, float*, int, int, int, void*);
typedef int (*ShapeFn)(const void*, int, int, int, int*, int*, int*);
typedef int (*ChainFn)(const void*, const float*, float*, int, int, int, void*, size_t, float* const*, void*);
typedef int (*StaticFn)(const void*, const float*, float*, int, int, int, float* const*, void*);
LayerFn g_layer[2];
ShapeFn g_shape;
ChainFn g_chain;
StaticFn g_static;
PyObject *g_handle, *g_dims, *g_c_in;

// A tensor that has memory of its own kind: no subclass, no wrapper of a transform.
const at::Tensor* plain(PyObject* o)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || t.layout() != at::kStrided || !t.device().is_cuda() || !t.has_storage() ||
        t.key_set().has_any(c10::DispatchKeySet({c10::DispatchKey::Python, c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::Batched,
                                                 c10::DispatchKey::FuncTorchGradWrapper, c10::DispatchKey::Functionalize,
                                                 c10::DispatchKey::ZeroTensor})))
        return nullptr;
    return &t;
}
const at::Tensor* activations(PyObject* o)
{
    const at::Tensor* t = plain(o);
    return t && t->scalar_type() == at::kFloat && t->is_contiguous() ? t : nullptr;
}
bool as_int(PyObject* o, int* v)
{
    if (!PyLong_CheckExact(o)) return false;
    int over = 0;
    const long l = PyLong_AsLongAndOverflow(o, &over);
    if (over || l < INT_MIN || l > INT_MAX) return false;
    *v = (int)l;
    return true;
}
void* handle_of(PyObject* p)
{
    PyObject* h = PyObject_GetAttr(p, g_handle);
    void* v = h && PyLong_CheckExact(h) ? PyLong_AsVoidPtr(h) : nullptr;
    Py_XDECREF(h);
    return v;
}
bool fits(const at::Tensor& t, long long pixels, long long channels)
{
    long long need = 0;
    return !__builtin_mul_overflow(pixels, channels, &need) && t.numel() >= need;
}
bool extents(PyObject* const* a, int (&e)[3])
{
    return as_int(a[0], &e[0]) && as_int(a[1], &e[1]) && as_int(a[2], &e[2]) && e[0] > 0 && e[1] > 0 && e[2] > 0;
}
// The body of a call: a result code of the library, or kOther.
constexpr long kOther = LONG_MIN;
template <class F>
PyObject* answer(F&& body)
{
    long rc = kOther;
    try {
        rc = body();
    } catch (...) {
        rc = kOther;
    }
    if (rc == kOther) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    return PyLong_FromLong(rc);
}

// layer(kind index, packed, x, y, n, h, w, stream)
PyObject* layer(PyObject*, PyObject* const* a, Py_ssize_t count)
{
    return answer([&]() -> long {
        int k, e[3];
        if (count != 8 || a[7] != Py_None || !as_int(a[0], &k) || k < 0 || k > 1 || !extents(a + 4, e)) return kOther;
        const at::Tensor *x = activations(a[2]), *y = activations(a[3]);
        if (!x || !y) return kOther;
        PyObject* d = PyObject_GetAttr(a[1], g_dims);                    // (c_in, c_out, stride), kept with the handle
        if (!d) return kOther;
        int c_in = 0, c_out = 0, stride = 0;
        const bool ok = PyTuple_CheckExact(d) && PyTuple_GET_SIZE(d) == 3 && as_int(PyTuple_GET_ITEM(d, 0), &c_in) &&
                        as_int(PyTuple_GET_ITEM(d, 1), &c_out) && as_int(PyTuple_GET_ITEM(d, 2), &stride) && stride > 0;
        Py_DECREF(d);
        void* const p = handle_of(a[1]);
        if (!ok || !p) return kOther;
        const int oh = k ? (e[1] - 1) / stride + 1 : e[1], ow = k ? (e[2] - 1) / stride + 1 : e[2];
        if ((long long)e[1] * e[2] > LLONG_MAX / e[0] || !fits(*x, (long long)e[1] * e[2] * e[0], c_in) ||
            !fits(*y, (long long)oh * ow * e[0], c_out))
            return kOther;
        const float* const xp = (const float*)x->data_ptr();
        float* const yp = (float*)y->data_ptr();
        void* const st = (void*)c10::hip::getCurrentHIPStream().stream();
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = g_layer[k](p, xp, yp, e[0], e[1], e[2], st);
        Py_END_ALLOW_THREADS
        return rc;
    });
}

// chain(chain, x, y, n, h, w, workspace or None for the built-in one, stream)
PyObject* chain(PyObject*, PyObject* const* a, Py_ssize_t count)
{
    return answer([&]() -> long {
        int e[3], oh, ow, oc, c_in = 0;
        if (count != 8 || a[7] != Py_None || !extents(a + 3, e)) return kOther;
        const at::Tensor *x = activations(a[1]), *y = activations(a[2]), *ws = a[6] == Py_None ? nullptr : plain(a[6]);
        void* const c = handle_of(a[0]);
        if (!x || !y || !c || (a[6] != Py_None && !ws)) return kOther;
        PyObject* ci = PyObject_GetAttr(a[0], g_c_in);
        const bool ok = ci && as_int(ci, &c_in);
        Py_XDECREF(ci);
        if (!ok || (long long)e[1] * e[2] > LLONG_MAX / e[0] || g_shape(c, e[0], e[1], e[2], &oh, &ow, &oc) != 0 ||
            !fits(*x, (long long)e[1] * e[2] * e[0], c_in) || !fits(*y, (long long)oh * ow * e[0], oc))
            return kOther;
        const float* const xp = (const float*)x->data_ptr();
        float* const yp = (float*)y->data_ptr();
        void* const wp = ws ? ws->data_ptr() : nullptr;
        const size_t bytes = ws ? (size_t)ws->numel() * ws->element_size() : 0;
        void* const st = (void*)c10::hip::getCurrentHIPStream().stream();
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = ws ? g_chain(c, xp, yp, e[0], e[1], e[2], wp, bytes, nullptr, st) : g_static(c, xp, yp, e[0], e[1], e[2], nullptr, st);
        Py_END_ALLOW_THREADS
        return rc;
    });
}

// bind(addresses of sbn_conv1x1_sparse, sbn_conv3x3_sparse, sbn_chain_output_shape, sbn_pointwise_chain, sbn_pointwise_chain_static)
PyObject* bind(PyObject*, PyObject* args)
{
    Py_ssize_t f[5];
    if (!PyArg_ParseTuple(args, "nnnnn", &f[0], &f[1], &f[2], &f[3], &f[4])) return nullptr;
    g_layer[0] = (LayerFn)f[0], g_layer[1] = (LayerFn)f[1], g_shape = (ShapeFn)f[2], g_chain = (ChainFn)f[3], g_static = (StaticFn)f[4];
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"layer", (PyCFunction)(void*)layer, METH_FASTCALL, nullptr},
                         {"chain", (PyCFunction)(void*)chain, METH_FASTCALL, nullptr},
                         {"bind", bind, METH_VARARGS, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal()
{
    g_handle = PyUnicode_InternFromString("handle");
    g_dims = PyUnicode_InternFromString("_dims");
    g_c_in = PyUnicode_InternFromString("c_in");
    return g_handle && g_dims && g_c_in ? PyModule_Create(&module) : nullptr;
}
