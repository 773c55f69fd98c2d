// marshal.cpp -- the short way from torch tensors to the C entry points, for the ordinary call.
//
// A call of the binding spends 9 us in Python besides the 3.6 us of the C entry point itself (attribute look-ups,
// two allocations, the current stream, ctypes conversions), which is more than the kernels of a small call take.  The
// functions here do the same for a call whose arguments are plain contiguous tensors on one GPU, and return None for
// every other one without having done anything: the binding's Python code then handles it, errors included.  Host
// only; the entry points' addresses come from the binding (set_entries), so nothing links to the library.
#include <ATen/ATen.h>
#include <Python.h>
#include <c10/core/DeviceGuard.h>
#include <pybind11/gil.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <climits>
#include <cmath>

namespace {

typedef int (*FwdFn)(const void *, const void *, const void *, void *, float *, int, int, int, int, int, int, float, void *);
typedef int (*SplitFn)(const void *, const void *, const void *, void *, float *, void *, long long, int, int, int, int, int,
                       int, int, float, void *);
typedef int (*BwdFn)(const void *, const void *, const void *, const void *, const void *, const float *, void *, void *,
                     void *, float *, int, int, int, int, int, int, float, void *);
typedef long long (*WsFn)(int, int, int, int, int);

// [0] bf16, [1] fp16
FwdFn g_fwd[2];
SplitFn g_split[2];
BwdFn g_bwd[2];
WsFn g_ws;
PyObject *g_current_stream;   // device index -> address of its current stream

const at::ScalarType kElem[2] = {at::kBFloat16, at::kHalf};

// a plain contiguous GPU tensor of this type (no subclass, nothing without memory of its own)
const at::Tensor *plain(PyObject *o, at::ScalarType type, int64_t dims)
{
    if (!THPVariable_CheckExact(o))
        return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || !t.has_storage() || t.scalar_type() != type ||
        (dims && t.dim() != dims) || !t.is_contiguous() || t.is_conj() || t.is_neg())
        return nullptr;
    return &t;
}

struct Shape {
    int B, H, S_q, S_kv, D;
};

bool same_shape(const at::Tensor &a, const at::Tensor &b) { return a.sizes() == b.sizes() && a.device() == b.device(); }

// q [B,H,S_q,D], k and v [B,H,S_kv,D] on one device, sizes the entry points can count
bool qkv(PyObject *const *a, at::ScalarType type, const at::Tensor *t[3], Shape &s)
{
    for (int i = 0; i < 3; ++i)
        if (!(t[i] = plain(a[i], type, 4)))
            return false;
    const auto q = t[0]->sizes(), k = t[1]->sizes();
    if (!same_shape(*t[1], *t[2]) || t[0]->device() != t[1]->device() || k[0] != q[0] || k[1] != q[1] || k[3] != q[3])
        return false;
    for (int i = 0; i < 4; ++i)
        if (q[i] < 1 || k[i] < 1 || q[i] > INT_MAX || k[i] > INT_MAX)
            return false;
    s = {(int)q[0], (int)q[1], (int)q[2], (int)k[2], (int)q[3]};
    return true;
}

bool is_lse(const at::Tensor &t, const Shape &s, const at::Tensor &q)
{
    return t.size(0) == s.B && t.size(1) == s.H && t.size(2) == s.S_q && t.device() == q.device();
}

bool scale_of(PyObject *o, int D, float &scale)
{
    if (o == Py_None)
        scale = (float)(1.0 / std::pow((double)D, 0.5));
    else if (PyFloat_CheckExact(o))
        scale = (float)PyFloat_AS_DOUBLE(o);
    else
        return false;
    return true;
}

// the address in a Python int (the reference is taken over)
bool address_of(PyObject *h, void *&address)
{
    address = h && PyLong_CheckExact(h) ? PyLong_AsVoidPtr(h) : nullptr;
    const bool ok = h && PyLong_CheckExact(h) && !PyErr_Occurred();
    Py_XDECREF(h);
    PyErr_Clear();
    return ok;
}

// The stream to launch on: the device's current one, or the one the caller names.  `allocates`: the call has something to
// allocate, and what is allocated here belongs to the current stream; a call that needs memory of another stream goes the
// other way.
bool stream_of(PyObject *o, const c10::Device &dev, bool allocates, void *&stream)
{
    void *current = nullptr;
    if (o == Py_None || allocates) {
        PyObject *index = PyLong_FromLong(dev.index());
        const bool ok = address_of(index && g_current_stream ? PyObject_CallOneArg(g_current_stream, index) : nullptr, current);
        Py_XDECREF(index);
        if (!ok)
            return false;
        if (o == Py_None) {
            stream = current;
            return true;
        }
    }
    return address_of(PyObject_GetAttrString(o, "cuda_stream"), stream) && (!allocates || stream == current);
}

// one of these arguments is left for the call to allocate
bool any_none(PyObject *const *a, int n)
{
    for (int i = 0; i < n; ++i)
        if (a[i] == Py_None)
            return true;
    return false;
}

// the launch, with the tensors' device current and the interpreter lock released
template <typename F>
int launch(const c10::Device &dev, F f)
{
    const c10::OptionalDeviceGuard guard(dev);
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f();
    Py_END_ALLOW_THREADS
    return rc;
}

PyObject *pack(std::initializer_list<const at::Tensor *> ts)
{
    PyObject *r = PyTuple_New((Py_ssize_t)ts.size());
    Py_ssize_t i = 0;
    for (const at::Tensor *t : ts) {
        PyObject *w = r ? THPVariable_Wrap(*t) : nullptr;
        if (!w) {
            Py_XDECREF(r);
            return nullptr;
        }
        PyTuple_SET_ITEM(r, i++, w);
    }
    return r;
}

// An allocation, with the interpreter lock released as torch's own functions do it: it may wait for the device, and other
// threads of the program (host callbacks of queued work among them) must be able to run meanwhile.
template <typename F>
at::Tensor allocate(F make)
{
    const pybind11::gil_scoped_release no_gil;
    return make();
}

// an output the caller may have given: taken as it is, or allocated like `like`; false if it needs the other way
bool output(PyObject *given, const at::Tensor &like, at::Tensor &out)
{
    if (given == Py_None) {
        out = allocate([&] { return at::empty_like(like); });
        return true;
    }
    const at::Tensor *t = plain(given, like.scalar_type(), 0);
    if (!t || !same_shape(*t, like))
        return false;
    out = *t;
    return true;
}

bool lse_output(PyObject *given, const Shape &s, const at::Tensor &q, at::Tensor &out)
{
    if (given == Py_None) {
        out = allocate([&] { return at::empty({s.B, s.H, s.S_q}, q.options().dtype(at::kFloat)); });
        return true;
    }
    const at::Tensor *t = plain(given, at::kFloat, 3);
    if (!t || !is_lse(*t, s, q))
        return false;
    out = *t;
    return true;
}

// True / False, or a truth value another object would have to be asked for
int truth(PyObject *o) { return o == Py_True ? 1 : o == Py_False ? 0 : -1; }

// 0 for bf16, 1 for fp16
int type_of(PyObject *o) { return (int)PyLong_AsLong(o) & 1; }

// fwd(type, q, k, v, o, lse, causal, scale, stream) -> (o, lse), a status other than 0, or None
PyObject *py_fwd(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    const at::Tensor *t[3];
    Shape s;
    float scale;
    void *stream;
    at::Tensor o, lse;
    const int type = n == 9 ? type_of(a[0]) : 0, causal = n == 9 ? truth(a[6]) : -1;
    if (n != 9 || causal < 0 || !g_fwd[type] || !qkv(a + 1, kElem[type], t, s) || !scale_of(a[7], s.D, scale) ||
        !stream_of(a[8], t[0]->device(), any_none(a + 4, 2), stream) || !output(a[4], *t[0], o) || !lse_output(a[5], s, *t[0], lse))
        Py_RETURN_NONE;
    const int rc = launch(t[0]->device(), [&] {
        return g_fwd[type](t[0]->data_ptr(), t[1]->data_ptr(), t[2]->data_ptr(), o.data_ptr(), (float *)lse.data_ptr(), s.B,
                           s.H, s.S_q, s.S_kv, s.D, causal, scale, stream);
    });
    return rc ? PyLong_FromLong(rc) : pack({&o, &lse});
    END_HANDLE_TH_ERRORS
}

// splitkv(type, q, k, v, n_split, o, lse, workspace, causal, scale, stream)
PyObject *py_splitkv(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    const at::Tensor *t[3];
    Shape s;
    float scale;
    void *stream;
    at::Tensor o, lse, ws;
    const int type = n == 11 ? type_of(a[0]) : 0, causal = n == 11 ? truth(a[8]) : -1;
    if (n != 11 || causal < 0 || !g_split[type] || !g_ws || !PyLong_CheckExact(a[4]) || !qkv(a + 1, kElem[type], t, s) ||
        !scale_of(a[9], s.D, scale) || !stream_of(a[10], t[0]->device(), any_none(a + 5, 3), stream))
        Py_RETURN_NONE;
    const long n_split = PyLong_AsLong(a[4]);
    if (PyErr_Occurred()) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    const long long need = n_split >= 1 && n_split <= 256 ? g_ws(s.B, s.H, s.S_q, s.D, (int)n_split) : -1;
    if (need < 1)
        Py_RETURN_NONE;
    if (a[7] != Py_None) {
        if (!THPVariable_CheckExact(a[7]))
            Py_RETURN_NONE;
        ws = THPVariable_Unpack(a[7]);
        if (!plain(a[7], ws.scalar_type(), 0) || ws.device() != t[0]->device())
            Py_RETURN_NONE;
    }
    if (!output(a[5], *t[0], o) || !lse_output(a[6], s, *t[0], lse))
        Py_RETURN_NONE;
    if (!ws.defined())
        ws = allocate([&] { return at::empty({need < 16 ? 16 : need}, t[0]->options().dtype(at::kByte)); });
    const int rc = launch(t[0]->device(), [&] {
        return g_split[type](t[0]->data_ptr(), t[1]->data_ptr(), t[2]->data_ptr(), o.data_ptr(), (float *)lse.data_ptr(),
                             ws.data_ptr(), (long long)ws.nbytes(), (int)n_split, s.B, s.H, s.S_q, s.S_kv, s.D, causal, scale,
                             stream);
    });
    return rc ? PyLong_FromLong(rc) : pack({&o, &lse});
    END_HANDLE_TH_ERRORS
}

// bwd(type, q, k, v, o, d_o, lse, dq, dk, dv, delta_ws, causal, scale, stream)
PyObject *py_bwd(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    const at::Tensor *t[3];
    Shape s;
    float scale;
    void *stream;
    at::Tensor g[3], ws;
    const int type = n == 14 ? type_of(a[0]) : 0, causal = n == 14 ? truth(a[11]) : -1;
    if (n != 14 || causal < 0 || !g_bwd[type] || !qkv(a + 1, kElem[type], t, s) || !scale_of(a[12], s.D, scale) ||
        !stream_of(a[13], t[0]->device(), any_none(a + 7, 4), stream))
        Py_RETURN_NONE;
    const at::Tensor *o = plain(a[4], kElem[type], 4), *d_o = plain(a[5], kElem[type], 4), *lse = plain(a[6], at::kFloat, 3);
    if (!o || !d_o || !lse || !same_shape(*o, *t[0]) || !same_shape(*d_o, *t[0]) || !is_lse(*lse, s, *t[0]))
        Py_RETURN_NONE;
    const int64_t rows2 = 2ll * s.B * s.H * s.S_q;
    if (a[10] != Py_None) {
        const at::Tensor *w = plain(a[10], at::kFloat, 0);
        if (!w || w->numel() < rows2 || w->device() != t[0]->device())
            Py_RETURN_NONE;
        ws = *w;
    }
    for (int i = 0; i < 3; ++i)
        if (!output(a[7 + i], *t[i], g[i]))
            Py_RETURN_NONE;
    if (!ws.defined())
        ws = allocate([&] { return at::empty({rows2}, t[0]->options().dtype(at::kFloat)); });
    const int rc = launch(t[0]->device(), [&] {
        return g_bwd[type](t[0]->data_ptr(), t[1]->data_ptr(), t[2]->data_ptr(), o->data_ptr(), d_o->data_ptr(),
                           (const float *)lse->data_ptr(), g[0].data_ptr(), g[1].data_ptr(), g[2].data_ptr(),
                           (float *)ws.data_ptr(), s.B, s.H, s.S_q, s.S_kv, s.D, causal, scale, stream);
    });
    return rc ? PyLong_FromLong(rc) : pack({&g[0], &g[1], &g[2]});
    END_HANDLE_TH_ERRORS
}

// set_entries(addresses of fwd bf16, fwd fp16, splitkv bf16, splitkv fp16, bwd bf16, bwd fp16, workspace size; then the
// function that returns a device's current stream)
PyObject *py_set_entries(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    void *p[7];
    if (n != 8 || !PyCallable_Check(a[7])) {
        PyErr_SetString(PyExc_TypeError, "set_entries takes seven addresses and a function");
        return nullptr;
    }
    for (int i = 0; i < 7; ++i)
        p[i] = PyLong_AsVoidPtr(a[i]);
    if (PyErr_Occurred())
        return nullptr;
    for (int i = 0; i < 2; ++i) {
        g_fwd[i] = (FwdFn)p[i];
        g_split[i] = (SplitFn)p[2 + i];
        g_bwd[i] = (BwdFn)p[4 + i];
    }
    g_ws = (WsFn)p[6];
    Py_INCREF(a[7]);
    Py_XSETREF(g_current_stream, a[7]);
    Py_RETURN_NONE;
}

PyMethodDef kMethods[] = {
    {"fwd", (PyCFunction)(void (*)(void))py_fwd, METH_FASTCALL, nullptr},
    {"splitkv", (PyCFunction)(void (*)(void))py_splitkv, METH_FASTCALL, nullptr},
    {"bwd", (PyCFunction)(void (*)(void))py_bwd, METH_FASTCALL, nullptr},
    {"set_entries", (PyCFunction)(void (*)(void))py_set_entries, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, kMethods};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) { return PyModule_Create(&kModule); }
