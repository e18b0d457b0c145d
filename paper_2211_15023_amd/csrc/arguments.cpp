// Argument marshalling of a policy's forwards, V-trace and the KL indicators, as a CPython module: tensors are checked and taken to pointers here, and
// the library is called without the interpreter's lock.  A call of 32 states on the 64-unit MLP costs the host what the checks, the
// conversions of eight ctypes arguments and the launch cost; the kernel takes 2.5 us.
//
// Every function returns the library's status, or None for arguments that are not plain: tensors of another type than torch.Tensor itself,
// another dtype, device or layout than the call takes, shapes that do not match, an active torch-function mode, a stream object.  The
// caller then goes the general way (binding.py), which raises the error or finds the pointer.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "accerl.h"

namespace {

PyTypeObject* handle_type = nullptr;      // ctypes.c_void_p
PyObject* value_name = nullptr;

// One argument after the other; `plain` turns false at the first one that is not.
struct Args {
    PyObject* const* at;
    bool plain;

    explicit Args(PyObject* const* a) : at(a), plain(!at::impl::torch_function_mode_enabled()) {}

    const at::Tensor* tensor() {
        PyObject* o = *at++;
        if (!plain || Py_TYPE(o) != (PyTypeObject*)THPVariableClass) { plain = false; return nullptr; }
        const at::Tensor& t = THPVariable_Unpack(o);
        if (!t.is_cuda() || !t.is_contiguous()) plain = false;
        return &t;
    }
    void* pointer(c10::ScalarType type) {
        if (*at == Py_None) { ++at; return nullptr; }
        const at::Tensor* t = tensor();
        if (plain && t->scalar_type() != type) plain = false;
        return plain ? t->data_ptr() : nullptr;
    }
    // a tensor of this shape
    void* shaped(c10::ScalarType type, c10::IntArrayRef shape) {
        const at::Tensor* t = tensor();
        if (plain && (t->scalar_type() != type || t->sizes() != shape)) plain = false;
        return plain ? t->data_ptr() : nullptr;
    }
    float* f32() { return (float*)pointer(c10::kFloat); }
    accerl_policy* handle() {
        PyObject* o = *at++;
        if (!plain || Py_TYPE(o) != handle_type) { plain = false; return nullptr; }
        PyObject* v = PyObject_GetAttr(o, value_name);
        void* p = v && v != Py_None ? PyLong_AsVoidPtr(v) : nullptr;
        Py_XDECREF(v);
        return (accerl_policy*)p;
    }
    void* states(int64_t* B) {
        const at::Tensor* t = tensor();
        if (plain && t->dim() < 1) plain = false;
        if (!plain) return nullptr;
        *B = t->size(0);
        return t->data_ptr();
    }
    void* stream() {
        PyObject* o = *at++;
        if (o == Py_None) return plain ? (void*)c10::hip::getCurrentHIPStream().stream() : nullptr;
        if (!PyLong_CheckExact(o)) { plain = false; return nullptr; }
        return PyLong_AsVoidPtr(o);
    }
    double number() {
        PyObject* o = *at++;
        if (!PyFloat_CheckExact(o)) { plain = false; return 0.0; }
        return PyFloat_AS_DOUBLE(o);
    }
};

// count arguments: parse(args) reads them in order and returns the call that is then made
template <class Parse>
PyObject* call(PyObject* const* argv, Py_ssize_t given, Py_ssize_t count, Parse&& parse) {
    if (given != count) { PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", count, given); return nullptr; }
    try {
        Args a(argv);
        auto made = parse(a);
        if (PyErr_Occurred()) { PyErr_Clear(); a.plain = false; }
        if (!a.plain) Py_RETURN_NONE;
        int rc = 0;
        bool threw = false;                      // (said only when the lock is held again, and never taken for arguments that are not plain)
        Py_BEGIN_ALLOW_THREADS
        try { rc = made(); } catch (...) { threw = true; }
        Py_END_ALLOW_THREADS
        if (threw) { PyErr_SetString(PyExc_RuntimeError, "the library threw an exception"); return nullptr; }
        return PyLong_FromLong(rc);
    } catch (const std::exception&) {            // a tensor without storage, for one: the general way says it
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

template <int (*F)(accerl_policy*, const void*, int64_t, const float*, float*, float*, int32_t*, void*)>
PyObject* forward(PyObject*, PyObject* const* argv, Py_ssize_t n) {
    return call(argv, n, 7, [](Args& a) {
        int64_t B = 0;
        accerl_policy* p = a.handle();
        void* x = a.states(&B);
        float *u = a.f32(), *l = a.f32(), *v = a.f32();
        int32_t* act = (int32_t*)a.pointer(c10::kInt);
        void* s = a.stream();
        return [=] { return F(p, x, B, u, l, v, act, s); };
    });
}

PyObject* recurrent(PyObject*, PyObject* const* argv, Py_ssize_t n) {
    return call(argv, n, 10, [](Args& a) {
        int64_t B = 0;
        accerl_policy* p = a.handle();
        void* x = a.states(&B);
        float* u = a.f32();
        uint8_t* done = (uint8_t*)a.pointer(c10::kByte);
        float *h = a.f32(), *c = a.f32(), *l = a.f32(), *v = a.f32();
        int32_t* act = (int32_t*)a.pointer(c10::kInt);
        void* s = a.stream();
        return [=] { return accerl_actor_forward_recurrent(p, x, B, u, done, h, c, l, v, act, s); };
    });
}

template <int (*F)(const float*, const float*, int64_t, int32_t, float*, float*, double*, void*)>
PyObject* monitor(PyObject*, PyObject* const* argv, Py_ssize_t n) {
    return call(argv, n, 6, [](Args& a) {
        const at::Tensor* o = a.tensor();
        if (a.plain && (o->scalar_type() != c10::kFloat || o->dim() != 2)) a.plain = false;
        const int64_t B = a.plain ? o->size(0) : 0, A = a.plain ? o->size(1) : 0;
        const float* po = a.plain ? (const float*)o->data_ptr() : nullptr;
        const float* ps = (const float*)a.shaped(c10::kFloat, {B, A});
        float *kl = a.f32(), *ent = a.f32();
        double* st = (double*)a.pointer(c10::kDouble);
        void* s = a.stream();
        return [=] { return F(po, ps, B, (int32_t)A, kl, ent, st, s); };
    });
}

PyObject* vtrace(PyObject*, PyObject* const* argv, Py_ssize_t n) {
    return call(argv, n, 13, [](Args& a) {
        const at::Tensor* o = a.tensor();
        if (a.plain && (o->scalar_type() != c10::kFloat || o->dim() != 3)) a.plain = false;
        const int64_t T = a.plain ? o->size(0) : 0, B = a.plain ? o->size(1) : 0, A = a.plain ? o->size(2) : 0;
        const float* po = a.plain ? (const float*)o->data_ptr() : nullptr;
        const float* ps = (const float*)a.shaped(c10::kFloat, {T, B, A});
        const int32_t* act = (const int32_t*)a.shaped(c10::kInt, {T, B});
        const float *rew = (const float*)a.shaped(c10::kFloat, {T, B}), *disc = (const float*)a.shaped(c10::kFloat, {T, B});
        const float* val = (const float*)a.shaped(c10::kFloat, {T, B});
        const float* boot = a.f32();
        const double rho_bar = a.number(), c_bar = a.number();
        float* vs = (float*)a.shaped(c10::kFloat, {T, B});
        float* adv = a.f32();
        float* rho = (float*)a.shaped(c10::kFloat, {T, B});
        void* s = a.stream();
        return [=] { return accerl_vtrace(po, ps, act, rew, disc, val, boot, T, B, (int32_t)A, (float)rho_bar, (float)c_bar, vs, adv, rho, s); };
    });
}

PyObject* init(PyObject*, PyObject* type) {
    if (!PyType_Check(type)) { PyErr_SetString(PyExc_TypeError, "expected ctypes.c_void_p"); return nullptr; }
    Py_INCREF(type);
    handle_type = (PyTypeObject*)type;
    Py_RETURN_NONE;
}

#define FAST(f) (PyCFunction)(void (*)(void))(f), METH_FASTCALL, nullptr
PyMethodDef methods[] = {
    {"init", init, METH_O, nullptr},
    {"forward", FAST(forward<accerl_actor_forward>)},
    {"forward_teacher", FAST(forward<accerl_actor_forward_teacher>)},
    {"forward_recurrent", FAST(recurrent)},
    {"monitor_kl", FAST(monitor<accerl_monitor_kl>)},
    {"monitor_kl_noalloc", FAST(monitor<accerl_monitor_kl_noalloc>)},
    {"vtrace", FAST(vtrace)},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "accerl_args", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_accerl_args() {
    value_name = PyUnicode_InternFromString("value");
    return value_name ? PyModule_Create(&module) : nullptr;
}
