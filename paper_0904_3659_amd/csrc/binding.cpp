// Native front of the two calls that small systems make most, nbody_forces and
// nbody_forces_backward: the checks of nbody.py, the result tensors and the C
// call without the interpreter in between.  Anything but the common case
// (plain contiguous float32 HIP tensors of the right shapes, a float eps2, no
// tensor subclass, wrapper or active function mode) returns None, and the
// Python code in nbody.py takes the call and names what is wrong.
//
// At 1,024 bodies a call from Python took 8.2 us (adjoint 8.8) for 2.7 us
// (3.6) of GPU work: four tensor checks, two torch.empty and a nine-argument
// ctypes call in the interpreter.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cmath>
#include <cstdint>
#include <new>

namespace {

using ForcesEx = int (*)(const float *, const float *, int64_t, float, float *, float *, uint32_t,
                         void *);
using Backward = int (*)(const float *, const float *, int64_t, float, const float *, const float *,
                         float *, float *, void *);
ForcesEx g_forces = nullptr;
Backward g_backward = nullptr;
PyObject *g_raw_stream = nullptr;  // torch._C._cuda_getCurrentRawStream

constexpr c10::DispatchKeySet kWrappers({c10::DispatchKey::Python, c10::DispatchKey::PythonTLSSnapshot,
                                         c10::DispatchKey::FuncTorchBatched,
                                         c10::DispatchKey::FuncTorchGradWrapper,
                                         c10::DispatchKey::Functionalize,
                                         c10::DispatchKey::Conjugate, c10::DispatchKey::Negative,
                                         c10::DispatchKey::ZeroTensor, c10::DispatchKey::Fake});

// The plain tensor behind o if it is a contiguous float32 HIP tensor of shape
// [n] (cols == 0) or [n, cols], else NULL; n < 0 takes any n.
const at::Tensor *plain(PyObject *o, int64_t n, int64_t cols)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.scalar_type() != at::kFloat ||
        t.layout() != at::kStrided || t.key_set().has_any(kWrappers) || !t.is_contiguous())
        return nullptr;
    if (t.dim() != (cols ? 2 : 1) || (cols && t.size(1) != cols) || (n >= 0 && t.size(0) != n))
        return nullptr;
    return &t;
}

bool plain_eps2(PyObject *o, float *out)
{
    if (!PyFloat_CheckExact(o)) return false;
    const double e = PyFloat_AS_DOUBLE(o);
    if (!(e >= 0.0) || std::isinf(e)) return false;
    *out = (float)e;
    return true;
}

// torch's current stream on device `index` (false with a Python error set).
bool current_stream(int index, void **stream)
{
    PyObject *i = PyLong_FromLong(index);
    if (!i) return false;
    PyObject *r = PyObject_CallOneArg(g_raw_stream, i);
    Py_DECREF(i);
    if (!r) return false;
    *stream = PyLong_AsVoidPtr(r);
    Py_DECREF(r);
    return !(*stream == nullptr && PyErr_Occurred());
}

// (a, b) as Python tensors; b may be undefined (None).
PyObject *pair_of(const at::Tensor &a, const at::Tensor &b)
{
    PyObject *pa = THPVariable_Wrap(a);
    PyObject *pb = b.defined() ? THPVariable_Wrap(b) : Py_NewRef(Py_None);
    if (!pa || !pb) {
        Py_XDECREF(pa);
        Py_XDECREF(pb);
        return nullptr;
    }
    PyObject *r = PyTuple_New(2);
    if (!r) return nullptr;
    PyTuple_SET_ITEM(r, 0, pa);
    PyTuple_SET_ITEM(r, 1, pb);
    return r;
}

// The result tensors of a call: those of `out` (None, or a tuple of a vector
// array and a scalar array or None) or new ones, the scalar one if `scalar` is
// true (looked at only here, as in nbody.py).  False: not the common case, or a
// Python error is set.
bool results(PyObject *out, int64_t n, PyObject *scalar, const at::Tensor &like, at::Tensor *v,
             at::Tensor *s)
{
    if (out == Py_None) {
        const int with = PyObject_IsTrue(scalar);
        if (with < 0) return false;
        *v = at::empty({n, 3}, like.options().requires_grad(false));
        if (with) *s = at::empty({n}, like.options().requires_grad(false));
        return true;
    }
    if (!PyTuple_CheckExact(out) || PyTuple_GET_SIZE(out) != 2) return false;
    const at::Tensor *a = plain(PyTuple_GET_ITEM(out, 0), n, 3);
    if (!a) return false;
    *v = *a;
    if (PyTuple_GET_ITEM(out, 1) != Py_None) {
        const at::Tensor *b = plain(PyTuple_GET_ITEM(out, 1), n, 0);
        if (!b) return false;
        *s = *b;
    }
    return true;
}

float *data(const at::Tensor &t) { return t.defined() ? static_cast<float *>(t.data_ptr()) : nullptr; }

// None for a call left to the Python code, or the Python error that is set.
PyObject *declined()
{
    if (PyErr_Occurred()) return nullptr;
    Py_RETURN_NONE;
}

// torch's C++ exceptions as the Python ones its own calls raise
// (torch.OutOfMemoryError where an array cannot be had).
template <class F>
PyObject *guarded(F f)
{
    HANDLE_TH_ERRORS
    return f();
    END_HANDLE_TH_ERRORS
}

// forces(x, m, eps2, out, potential, flags) -> (a, p or None), a status != 0,
// or None
PyObject *forces(PyObject *, PyObject *const *args, Py_ssize_t count)
{
    return guarded([&]() -> PyObject * {
        if (count != 6 || !g_forces || at::impl::torch_function_mode_enabled()) Py_RETURN_NONE;
        float eps2;
        const at::Tensor *x = plain(args[0], -1, 3);
        const at::Tensor *m = x ? plain(args[1], x->size(0), 0) : nullptr;
        if (!m || !plain_eps2(args[2], &eps2)) Py_RETURN_NONE;
        const int64_t n = x->size(0);
        at::Tensor a, p;
        if (!results(args[3], n, args[4], *x, &a, &p)) return declined();
        void *stream;
        if (!current_stream(x->get_device(), &stream)) return nullptr;
        const uint32_t flags = (uint32_t)PyLong_AsUnsignedLong(args[5]);
        float *px = data(*x), *pm = data(*m), *pa = data(a), *pp = data(p);
        int status;
        Py_BEGIN_ALLOW_THREADS;
        status = g_forces(px, pm, n, eps2, pa, pp, flags, stream);
        Py_END_ALLOW_THREADS;
        return status ? PyLong_FromLong(status) : pair_of(a, p);
    });
}

// backward(x, m, eps2, grad_a, grad_p, need_grad_m, out)
PyObject *backward(PyObject *, PyObject *const *args, Py_ssize_t count)
{
    return guarded([&]() -> PyObject * {
        if (count != 7 || !g_backward || at::impl::torch_function_mode_enabled()) Py_RETURN_NONE;
        float eps2;
        const at::Tensor *x = plain(args[0], -1, 3);
        const at::Tensor *m = x ? plain(args[1], x->size(0), 0) : nullptr;
        if (!m || !plain_eps2(args[2], &eps2)) Py_RETURN_NONE;
        const int64_t n = x->size(0);
        const at::Tensor none;
        const at::Tensor *ga = args[3] == Py_None ? &none : plain(args[3], n, 3);
        const at::Tensor *gp = args[4] == Py_None ? &none : plain(args[4], n, 0);
        if (!ga || !gp) Py_RETURN_NONE;
        at::Tensor gx, gm;
        if (!results(args[6], n, args[5], *x, &gx, &gm)) return declined();
        void *stream;
        if (!current_stream(x->get_device(), &stream)) return nullptr;
        float *px = data(*x), *pm = data(*m), *pga = data(*ga), *pgp = data(*gp);
        float *pgx = data(gx), *pgm = data(gm);
        int status;
        Py_BEGIN_ALLOW_THREADS;
        status = g_backward(px, pm, n, eps2, pga, pgp, pgx, pgm, stream);
        Py_END_ALLOW_THREADS;
        return status ? PyLong_FromLong(status) : pair_of(gx, gm);
    });
}

// A forces call on fixed arrays (BoundForces): prepared once, then only the
// current stream is looked up per call.
struct Prepared {
    const float *x, *m;
    int64_t n;
    float eps2;
    float *a, *p;
    int device;
};
constexpr const char *kPrepared = "nbody prepared forces";

void drop(PyObject *capsule) { delete static_cast<Prepared *>(PyCapsule_GetPointer(capsule, kPrepared)); }

// prepare(x, m, n, eps2, a, p, device index): addresses as integers, p 0 for
// none; the caller has checked the tensors and keeps them
PyObject *prepare(PyObject *, PyObject *args)
{
    unsigned long long x, m, a, p;
    long long n;
    double eps2;
    int device;
    if (!PyArg_ParseTuple(args, "KKLdKKi", &x, &m, &n, &eps2, &a, &p, &device)) return nullptr;
    auto *c = new (std::nothrow) Prepared{
        reinterpret_cast<const float *>((uintptr_t)x), reinterpret_cast<const float *>((uintptr_t)m),
        (int64_t)n, (float)eps2, reinterpret_cast<float *>((uintptr_t)a),
        reinterpret_cast<float *>((uintptr_t)p), device};
    if (!c) return PyErr_NoMemory();
    PyObject *r = PyCapsule_New(c, kPrepared, drop);
    if (!r) delete c;
    return r;
}

// call(capsule) -> status
PyObject *call(PyObject *, PyObject *capsule)
{
    const auto *c = static_cast<const Prepared *>(PyCapsule_GetPointer(capsule, kPrepared));
    void *stream;
    if (!c || !current_stream(c->device, &stream)) return nullptr;
    int status;
    Py_BEGIN_ALLOW_THREADS;
    status = g_forces(c->x, c->m, c->n, c->eps2, c->a, c->p, 0u, stream);
    Py_END_ALLOW_THREADS;
    return PyLong_FromLong(status);
}

// bind(address of nbody_forces_ex, address of nbody_forces_backward,
//      torch._C._cuda_getCurrentRawStream)
PyObject *bind(PyObject *, PyObject *const *args, Py_ssize_t count)
{
    if (count != 3) {
        PyErr_SetString(PyExc_TypeError, "bind takes three arguments");
        return nullptr;
    }
    void *f = PyLong_AsVoidPtr(args[0]);
    void *b = PyLong_AsVoidPtr(args[1]);
    if (PyErr_Occurred()) return nullptr;
    PyObject *old = g_raw_stream;
    g_raw_stream = Py_NewRef(args[2]);
    Py_XDECREF(old);
    g_forces = reinterpret_cast<ForcesEx>(f);
    g_backward = reinterpret_cast<Backward>(b);
    Py_RETURN_NONE;
}

PyMethodDef kMethods[] = {
    {"bind", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(bind)), METH_FASTCALL, nullptr},
    {"forces", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(forces)), METH_FASTCALL, nullptr},
    {"backward", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(backward)), METH_FASTCALL,
     nullptr},
    {"prepare", prepare, METH_VARARGS, nullptr},
    {"call", call, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, kMethods,
                       nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() { return PyModule_Create(&kModule); }
