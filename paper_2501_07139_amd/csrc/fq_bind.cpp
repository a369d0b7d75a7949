// The way from a Python call to its C entry point for the calls that a served token or a small linear makes: argument checks, device
// addresses and the current stream without a Python call each.  A call of fq_qlinear at 16 x 512 x 512 took 5.7 us through
// ctypes, 3.7 of them the launch itself; through here 4.0.
//
// Every function takes the arguments of its namesake in the package and returns the entry point's code, or None when
// something is not as the plain case has it (an output to allocate, another tensor type, a size that does not fit,
// a wrong type): the caller then goes the long way, which allocates or raises.  Nothing is kept from one call to the next.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "fq.h"

#include <climits>
#include <memory>

namespace {

// entry points of libfq, as the package has loaded it
struct Entries {
    decltype(&fq_qlinear_tile) qlinear;
    decltype(&fq_qlinear_mixed) mixed;
    decltype(&fq_dense_f16) dense;
    decltype(&fq_head_nll) head_nll;
    decltype(&fq_token_nll) token_nll;
    decltype(&fq_logit_l2) logit_l2;
} entry;

PyObject *s_packed, *s_scales, *s_zeros, *s_n, *s_k, *s_bits;

// A contiguous device tensor of plain type, else nullptr.
const at::Tensor *device_tensor(PyObject *o, at::ScalarType type)
{
    if (!THPVariable_CheckExact(o))
        return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    return t.is_cuda() && t.scalar_type() == type && t.is_contiguous() ? &t : nullptr;
}

const at::Tensor *half_matrix(PyObject *o, int *rows, int *cols)
{
    const at::Tensor *t = device_tensor(o, at::kHalf);
    if (!t || t->dim() != 2 || t->size(0) > INT_MAX || t->size(1) > INT_MAX)
        return nullptr;
    *rows = (int)t->size(0);
    *cols = (int)t->size(1);
    return t;
}

// None: the current stream; a number: that handle.
bool stream_of(PyObject *o, void **stream)
{
    if (o == Py_None) {
        *stream = c10::hip::getCurrentHIPStream().stream();
        return true;
    }
    if (!PyLong_CheckExact(o))
        return false;
    *stream = PyLong_AsVoidPtr(o);
    return !PyErr_Occurred();
}

bool int_of(PyObject *o, int *v)
{
    if (!PyLong_CheckExact(o))
        return false;
    int overflow = 0;
    const long l = PyLong_AsLongAndOverflow(o, &overflow);
    if (overflow || l < INT_MIN || l > INT_MAX)
        return false;
    *v = (int)l;
    return true;
}

bool int_attr(PyObject *o, PyObject *name, int *v)
{
    PyObject *a = PyObject_GetAttr(o, name);
    if (!a)
        return false;
    const bool ok = int_of(a, v);
    Py_DECREF(a);
    return ok;
}

// Address of an attribute that is a tensor; the object keeps the tensor alive during the call.
bool tensor_attr(PyObject *o, PyObject *name, const void **v)
{
    PyObject *a = PyObject_GetAttr(o, name);
    if (!a)
        return false;
    const bool ok = THPVariable_CheckExact(a);
    if (ok)
        *v = THPVariable_Unpack(a).data_ptr();
    Py_DECREF(a);
    return ok;
}

bool matrix_of(PyObject *w, fq_segment *m, int *K)
{
    return tensor_attr(w, s_packed, &m->packed) && tensor_attr(w, s_scales, &m->scales) && tensor_attr(w, s_zeros, &m->zeros) &&
           int_attr(w, s_n, &m->N) && int_attr(w, s_k, K) && int_attr(w, s_bits, &m->bits);
}

// f(args) with C++ exceptions (a tensor without storage) and pending Python errors turned into "the long way".
template <class F>
PyObject *guarded(Py_ssize_t have, Py_ssize_t need, F &&f)
{
    int rc = 0;
    bool done = false;
    if (have == need) {
        try {
            done = f(&rc);
        } catch (...) {
            done = false;
        }
    }
    if (done)
        return PyLong_FromLong(rc);
    PyErr_Clear();
    Py_RETURN_NONE;
}

template <class F>
int without_gil(F &&f)
{
    int rc;
    Py_BEGIN_ALLOW_THREADS rc = f();
    Py_END_ALLOW_THREADS return rc;
}

PyObject *qlinear(PyObject *, PyObject *const *a, Py_ssize_t n) // x, w, out, stream, group, tile_rows
{
    return guarded(n, 6, [&](int *rc) {
        int M, K, wk, group, tile_rows;
        void *stream;
        fq_segment w;
        const at::Tensor *x = half_matrix(a[0], &M, &K), *out = device_tensor(a[2], at::kHalf);
        if (!x || !out || !matrix_of(a[1], &w, &wk) || wk != K || !stream_of(a[3], &stream) || !int_of(a[4], &group) ||
            !int_of(a[5], &tile_rows))
            return false;
        const void *px = x->data_ptr();
        void *po = out->data_ptr();
        *rc = without_gil([&] { return entry.qlinear(px, M, w.packed, w.scales, w.zeros, w.N, K, w.bits, group, po, tile_rows, stream); });
        return true;
    });
}

PyObject *mixed(PyObject *, PyObject *const *a, Py_ssize_t n) // x, segments (list or tuple), out, stream, group
{
    return guarded(n, 5, [&](int *rc) {
        int M, K, group;
        void *stream;
        fq_segment seg[FQ_MAX_SEGMENTS];
        const at::Tensor *x = half_matrix(a[0], &M, &K), *out = device_tensor(a[2], at::kHalf);
        if (!x || !out || !(PyList_CheckExact(a[1]) || PyTuple_CheckExact(a[1])) || !stream_of(a[3], &stream) || !int_of(a[4], &group))
            return false;
        // its items, held: reading an attribute may run Python code, which may change the list
        const std::unique_ptr<PyObject, void (*)(PyObject *)> items(PySequence_Tuple(a[1]), [](PyObject *o) { Py_DECREF(o); });
        const Py_ssize_t count = items ? PyTuple_GET_SIZE(items.get()) : 0;
        if (count < 1 || count > FQ_MAX_SEGMENTS)
            return false;
        for (Py_ssize_t i = 0; i < count; ++i) {
            int wk;
            if (!matrix_of(PyTuple_GET_ITEM(items.get(), i), &seg[i], &wk) || wk != K)
                return false;
        }
        const void *px = x->data_ptr();
        void *po = out->data_ptr();
        *rc = without_gil([&] { return entry.mixed(px, M, seg, (int)count, K, group, po, stream); });
        return true;
    });
}

PyObject *dense_f16(PyObject *, PyObject *const *a, Py_ssize_t n) // x, W, out, stream
{
    return guarded(n, 4, [&](int *rc) {
        int M, K, N, wk;
        void *stream;
        const at::Tensor *x = half_matrix(a[0], &M, &K), *W = half_matrix(a[1], &N, &wk), *out = device_tensor(a[2], at::kHalf);
        if (!x || !W || !out || wk != K || !stream_of(a[3], &stream))
            return false;
        const void *px = x->data_ptr(), *pw = W->data_ptr();
        void *po = out->data_ptr();
        *rc = without_gil([&] { return entry.dense(px, M, pw, N, K, po, stream); });
        return true;
    });
}

PyObject *head_nll(PyObject *, PyObject *const *a, Py_ssize_t n) // x, W, labels, out, workspace, stream
{
    return guarded(n, 6, [&](int *rc) {
        int M, K, V, wk;
        void *stream;
        const at::Tensor *x = half_matrix(a[0], &M, &K), *W = half_matrix(a[1], &V, &wk), *labels = device_tensor(a[2], at::kInt),
                         *out = device_tensor(a[3], at::kFloat), *ws = device_tensor(a[4], at::kByte);
        if (!x || !W || !labels || !out || !ws || wk != K || labels->numel() != M || !stream_of(a[5], &stream))
            return false;
        const void *px = x->data_ptr(), *pw = W->data_ptr();
        const int32_t *pl = static_cast<const int32_t *>(labels->data_ptr());
        float *po = static_cast<float *>(out->data_ptr());
        void *pws = ws->data_ptr();
        const size_t bytes = (size_t)ws->numel();
        *rc = without_gil([&] { return entry.head_nll(px, M, pw, V, K, pl, po, pws, bytes, stream); });
        return true;
    });
}

PyObject *token_nll(PyObject *, PyObject *const *a, Py_ssize_t n) // logits, labels, out, stream
{
    return guarded(n, 4, [&](int *rc) {
        int M, V;
        void *stream;
        const at::Tensor *l = half_matrix(a[0], &M, &V), *labels = device_tensor(a[1], at::kInt), *out = device_tensor(a[2], at::kFloat);
        if (!l || !labels || !out || !stream_of(a[3], &stream))
            return false;
        const void *pl = l->data_ptr();
        const int32_t *pi = static_cast<const int32_t *>(labels->data_ptr());
        float *po = static_cast<float *>(out->data_ptr());
        *rc = without_gil([&] { return entry.token_nll(pl, pi, M, V, po, stream); });
        return true;
    });
}

PyObject *logit_l2(PyObject *, PyObject *const *a, Py_ssize_t n) // a, b, out, stream
{
    return guarded(n, 4, [&](int *rc) {
        int M, V, mb, vb;
        void *stream;
        const at::Tensor *x = half_matrix(a[0], &M, &V), *y = half_matrix(a[1], &mb, &vb), *out = device_tensor(a[2], at::kFloat);
        if (!x || !y || !out || mb != M || vb != V || !stream_of(a[3], &stream))
            return false;
        const void *px = x->data_ptr(), *py = y->data_ptr();
        float *po = static_cast<float *>(out->data_ptr());
        *rc = without_gil([&] { return entry.logit_l2(px, py, M, V, po, stream); });
        return true;
    });
}

PyObject *bind(PyObject *, PyObject *args) // addresses of the entry points, in the order of Entries
{
    unsigned long long p[6];
    if (!PyArg_ParseTuple(args, "KKKKKK", &p[0], &p[1], &p[2], &p[3], &p[4], &p[5]))
        return nullptr;
    entry = Entries{reinterpret_cast<decltype(entry.qlinear)>(p[0]),  reinterpret_cast<decltype(entry.mixed)>(p[1]),
                    reinterpret_cast<decltype(entry.dense)>(p[2]),    reinterpret_cast<decltype(entry.head_nll)>(p[3]),
                    reinterpret_cast<decltype(entry.token_nll)>(p[4]), reinterpret_cast<decltype(entry.logit_l2)>(p[5])};
    Py_RETURN_NONE;
}

#define FQ_FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FQ_FAST(qlinear),   FQ_FAST(mixed),    FQ_FAST(dense_f16), FQ_FAST(head_nll),
                         FQ_FAST(token_nll), FQ_FAST(logit_l2), {"bind", bind, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_bind", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

} // namespace

PyMODINIT_FUNC PyInit__bind()
{
    s_packed = PyUnicode_InternFromString("packed");
    s_scales = PyUnicode_InternFromString("scales");
    s_zeros = PyUnicode_InternFromString("zeros");
    s_n = PyUnicode_InternFromString("N");
    s_k = PyUnicode_InternFromString("K");
    s_bits = PyUnicode_InternFromString("bits");
    PyObject *m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "torch_version", FQ_TORCH_VERSION) != 0) { // tensors are read by this version's layout
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
