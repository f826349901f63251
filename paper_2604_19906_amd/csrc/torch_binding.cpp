// The tensor functions of tpo.py as one native call each: the checks of the arguments, the output tensor and the library
// call.  On a small batch the Python form of the same steps takes longer than the kernel (a dozen attribute reads, a tuple of
// converted arguments): fp64 n = 7, 1000 elements, 6.4 us a call against 4.3 (calls whose kernel is
// shorter than the call 1.4 to 1.8 times as fast; a call that is waited for alone 18 against 22 us).
//
// Only the plain case is done here: exact torch.Tensor objects on a device, dense, without any wrapper or mode in their
// dispatch keys, outside of torch function modes (which see the Python form's calls, the new output's among them), arguments as
// documented.  For everything else a function returns None without having done anything, and the Python form takes the call with
// its own checks and errors.  A status other than TPO_OK comes back as a number.
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/ops/empty.h>
#include <ATen/ops/empty_like.h>
#include <c10/core/DispatchKeySet.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "tpo.h"

namespace {

struct Library {
    decltype(&tpo_ihelm_apply_variant) apply = nullptr;
    decltype(&tpo_ihelm_apply_sep_variant) sep = nullptr;
    decltype(&tpo_transform_apply) transform = nullptr;
    decltype(&tpo_convection_apply) convection = nullptr;
    decltype(&tpo_ihelm_apply_aniso) aniso = nullptr;
} lib;

// What a plain device tensor carries; anything more is a wrapper (vmap, functionalisation, a lazy conjugate, ..).
constexpr c10::DispatchKeySet kPlain({c10::DispatchKey::CUDA, c10::DispatchKey::AutogradCUDA, c10::DispatchKey::ADInplaceOrView,
                                      c10::DispatchKey::AutocastCUDA});

// The tensor behind an argument if it is a plain contiguous one, else null.
const at::Tensor *plain(PyObject *o)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || (t.key_set() | kPlain) != kPlain || !t.is_cuda() || !t.is_contiguous() || t.numel() == 0) return nullptr;
    return &t;
}

// `count` arguments as plain tensors of the first one's type; false if one is not, or if a torch function mode is active.
bool plain_all(PyObject *const *args, int count, const at::Tensor **out)
{
    if (at::impl::torch_function_mode_enabled()) return false;
    for (int k = 0; k < count; ++k) {
        int same = 0;
        while (same < k && args[same] != args[k]) ++same;
        out[k] = same < k ? out[same] : plain(args[k]);
        if (!out[k] || out[k]->scalar_type() != out[0]->scalar_type()) return false;
    }
    return true;
}

int dtype_code(const at::Tensor &t)
{
    return t.scalar_type() == at::kDouble ? TPO_F64 : t.scalar_type() == at::kFloat ? TPO_F32 : -1;
}
bool has_shape(const at::Tensor &t, std::initializer_list<int64_t> dims) { return t.sizes() == c10::IntArrayRef(dims); }

bool small_int(PyObject *o, int *value)
{
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    const long v = PyLong_AsLongAndOverflow(o, &overflow);
    if (overflow || v < 0 || v > 255) return false;
    *value = (int)v;
    return true;
}

// The output: the caller's tensor if it is plain and of that shape and type, a new one for None.
bool output(PyObject *o, const at::Tensor &like, c10::IntArrayRef dims, at::Tensor *out)
{
    if (o == Py_None) {
        *out = like.sizes() == dims ? at::empty_like(like) : at::empty(dims, like.options());
        return true;
    }
    const at::Tensor *t = plain(o);
    if (!t || t->scalar_type() != like.scalar_type() || t->sizes() != dims) return false;
    *out = *t;
    return true;
}

// Calls f(stream) without the interpreter lock and returns the output tensor or the status.
template <typename F>
PyObject *launch(PyObject *given, const at::Tensor &out, F &&f)
{
    void *stream = (void *)c10::hip::getCurrentHIPStream(c10::hip::current_device()).stream();
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = f(stream);
    Py_END_ALLOW_THREADS
    if (status != TPO_OK) return PyLong_FromLong(status);
    if (given == Py_None) return THPVariable_Wrap(out);
    Py_INCREF(given);
    return given;
}

// No C++ exception leaves a function: the call is declined instead.
template <typename F>
PyObject *guarded(F &&f)
{
    try {
        if (PyObject *r = f()) return r;
    } catch (...) {
    }
    if (PyErr_Occurred()) return nullptr;
    Py_RETURN_NONE;
}

// apply(u, S_x, S_y, S_z, D, v, variant), sizes along the axes as u has them
PyObject *cube(PyObject *const *args, Py_ssize_t n, bool cubic)
{
    return guarded([&]() -> PyObject * {
        const at::Tensor *t[5];
        int variant = TPO_VARIANT_AUTO;
        if (n != (cubic ? 7 : 6) || !plain_all(args, 5, t) || (cubic && !small_int(args[6], &variant))) return nullptr;
        const at::Tensor &u = *t[0];
        const int dt = dtype_code(u);
        if (dt < 0 || u.dim() != 4 || t[4]->sizes() != u.sizes()) return nullptr;
        const int64_t e = u.size(0), x = u.size(1), y = u.size(2), z = u.size(3);
        if (x > TPO_MAX_N || y > TPO_MAX_N || z > TPO_MAX_N || (cubic && (y != x || z != x))) return nullptr;
        if (!has_shape(*t[1], {x, x}) || !has_shape(*t[2], {y, y}) || !has_shape(*t[3], {z, z})) return nullptr;
        at::Tensor v;
        if (!output(args[5], u, u.sizes(), &v)) return nullptr;
        const void *p[5];
        for (int k = 0; k < 5; ++k) p[k] = t[k]->data_ptr();
        void *pv = v.data_ptr();
        return launch(args[5], v, [&](void *stream) {
            return cubic ? lib.apply(p[0], p[1], p[2], p[3], p[4], pv, (int)x, e, dt, stream, variant)
                         : lib.aniso(p[0], p[1], p[2], p[3], p[4], pv, (int)x, (int)y, (int)z, e, dt, stream);
        });
    });
}
PyObject *apply(PyObject *, PyObject *const *args, Py_ssize_t n) { return cube(args, n, true); }
PyObject *apply_aniso(PyObject *, PyObject *const *args, Py_ssize_t n) { return cube(args, n, false); }

// apply_sep(u, S_x, S_y, S_z, lam_x, lam_y, lam_z, mu, v, variant)
PyObject *apply_sep(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return guarded([&]() -> PyObject * {
        const at::Tensor *t[8];
        int variant;
        if (n != 10 || !plain_all(args, 8, t) || !small_int(args[9], &variant)) return nullptr;
        const at::Tensor &u = *t[0];
        const int dt = dtype_code(u);
        if (dt < 0 || u.dim() != 4) return nullptr;
        const int64_t e = u.size(0), m = u.size(1);
        if (m > TPO_MAX_N || u.size(2) != m || u.size(3) != m || !has_shape(*t[7], {e})) return nullptr;
        for (int k = 1; k < 4; ++k)
            if (!has_shape(*t[k], {m, m}) || !has_shape(*t[k + 3], {m})) return nullptr;
        at::Tensor v;
        if (!output(args[8], u, u.sizes(), &v)) return nullptr;
        const void *p[8];
        for (int k = 0; k < 8; ++k) p[k] = t[k]->data_ptr();
        void *pv = v.data_ptr();
        return launch(args[8], v, [&](void *stream) {
            return lib.sep(p[0], p[1], p[2], p[3], p[4], p[5], p[6], p[7], pv, (int)m, e, dt, stream, variant);
        });
    });
}

// transform(u, S_x, S_y, S_z, direction, t)
PyObject *transform(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return guarded([&]() -> PyObject * {
        const at::Tensor *t[4];
        int direction;
        if (n != 6 || !plain_all(args, 4, t) || !small_int(args[4], &direction)) return nullptr;
        const at::Tensor &u = *t[0];
        const int dt = dtype_code(u);
        if (dt < 0 || u.dim() != 4) return nullptr;
        const int64_t e = u.size(0), m = u.size(1);
        if (m > TPO_MAX_N || u.size(2) != m || u.size(3) != m) return nullptr;
        for (int k = 1; k < 4; ++k)
            if (!has_shape(*t[k], {m, m})) return nullptr;
        at::Tensor v;
        if (!output(args[5], u, u.sizes(), &v)) return nullptr;
        const void *p[4];
        for (int k = 0; k < 4; ++k) p[k] = t[k]->data_ptr();
        void *pv = v.data_ptr();
        return launch(args[5], v, [&](void *stream) {
            return lib.transform(p[0], p[1], p[2], p[3], pv, (int)m, e, dt, direction, stream);
        });
    });
}

// convection(P, M, D_vq, I_vq, F)
PyObject *convection(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return guarded([&]() -> PyObject * {
        const at::Tensor *t[4];
        if (n != 5 || !plain_all(args, 4, t)) return nullptr;
        const int dt = dtype_code(*t[0]);
        if (dt < 0 || t[2]->dim() != 2 || t[1]->dim() != 4) return nullptr;
        const int64_t v = t[2]->size(0), q = t[2]->size(1), e = t[1]->size(0);
        if (v > TPO_MAX_N || q > TPO_MAX_N || !has_shape(*t[3], {v, q}) || !has_shape(*t[1], {e, q, q, q})
            || !has_shape(*t[0], {3, 3, e, q, q, q}))
            return nullptr;
        at::Tensor f;
        if (!output(args[4], *t[0], {3, e, v, v, v}, &f)) return nullptr;
        const void *p[4];
        for (int k = 0; k < 4; ++k) p[k] = t[k]->data_ptr();
        void *pf = f.data_ptr();
        return launch(args[4], f, [&](void *stream) {
            return lib.convection(p[0], p[1], p[2], p[3], pf, (int)v, (int)q, e, dt, stream);
        });
    });
}

// bind(apply, sep, transform, convection, aniso): addresses of the library's functions
PyObject *bind(PyObject *, PyObject *args)
{
    unsigned long long a[5];
    if (!PyArg_ParseTuple(args, "KKKKK", &a[0], &a[1], &a[2], &a[3], &a[4])) return nullptr;
    lib.apply = reinterpret_cast<decltype(lib.apply)>(a[0]);
    lib.sep = reinterpret_cast<decltype(lib.sep)>(a[1]);
    lib.transform = reinterpret_cast<decltype(lib.transform)>(a[2]);
    lib.convection = reinterpret_cast<decltype(lib.convection)>(a[3]);
    lib.aniso = reinterpret_cast<decltype(lib.aniso)>(a[4]);
    Py_RETURN_NONE;
}

#define TPO_FAST(f) reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(&f)), METH_FASTCALL, nullptr
PyMethodDef methods[] = {
    {"apply", TPO_FAST(apply)},
    {"apply_aniso", TPO_FAST(apply_aniso)},
    {"apply_sep", TPO_FAST(apply_sep)},
    {"transform", TPO_FAST(transform)},
    {"convection", TPO_FAST(convection)},
    {"bind", &bind, METH_VARARGS, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_tpo_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// built_for: what this file was compiled against (binding_versions() in tpo.py), compared before any other use.  The accessors above are
// inlined with the offsets of that torch, so another one may well load and read the wrong members.
PyMODINIT_FUNC PyInit__tpo_torch(void)
{
    PyObject *m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "built_for", TPO_BUILT_FOR) < 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
