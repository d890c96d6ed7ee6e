// CPython front of the calls that a program issues once per operator: turns addresses and handles into the C ABI's arguments
// without a foreign-function layer in between (a call on a mini-batch costs about as much in Python as in the library:
// marshalling through ctypes took 1.1 us of the 4.1 us of a small Apply, here it takes 0.4).
//
// Every function takes plain integers (addresses of the ctypes structures that binding.py owns, table handles, device
// pointers; 0 or None = NULL), contiguous buffers of the stated item size where the ABI takes a host array, and the stream
// last: an integer handle, or None for torch's current stream.  A status other than DOL_OK goes to the error callback set
// with setup(), whose exception leaves the call.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstdint>

#include "dolphin_hip.h"

namespace {

PyObject *g_fail = nullptr, *g_device = nullptr, *g_stream = nullptr;

PyObject *done(dol_status st)
{
    if (st == DOL_OK) Py_RETURN_NONE;
    PyObject *code = PyLong_FromLong(st);
    PyObject *r = code ? PyObject_CallOneArg(g_fail, code) : nullptr;
    Py_XDECREF(code);
    return r;                               // (the callback raises)
}

// One call's arguments; `bad` once something did not convert (a Python error is set then).
struct Args {
    PyObject *const *v;
    bool bad = false;

    Args(PyObject *const *args, Py_ssize_t n, Py_ssize_t want) : v(args)
    {
        if (n != want) {
            PyErr_Format(PyExc_TypeError, "%zd arguments, %zd wanted", n, want);
            bad = true;
        }
    }
    template <typename T>
    T *ptr(int k)
    {
        if (bad || v[k] == Py_None) return nullptr;
        void *p = PyLong_AsVoidPtr(v[k]);
        if (!p && PyErr_Occurred()) bad = true;
        return static_cast<T *>(p);
    }
    int64_t num(int k)
    {
        if (bad) return 0;
        const long long x = PyLong_AsLongLong(v[k]);
        if (x == -1 && PyErr_Occurred()) bad = true;
        return x;
    }
    void *stream(int k)
    {
        if (bad) return nullptr;
        if (v[k] != Py_None) return ptr<void>(k);
        PyObject *dev = PyObject_CallNoArgs(g_device);
        PyObject *raw = dev ? PyObject_CallOneArg(g_stream, dev) : nullptr;
        Py_XDECREF(dev);
        void *p = raw ? PyLong_AsVoidPtr(raw) : nullptr;
        if (!raw || (!p && PyErr_Occurred())) bad = true;
        Py_XDECREF(raw);
        return p;
    }
};

// A contiguous host array for the time of a call.
struct Buffer {
    Py_buffer b{};
    bool held = false;

    Buffer(Args &a, int k)
    {
        if (a.bad) return;
        if (PyObject_GetBuffer(a.v[k], &b, PyBUF_SIMPLE) == 0) held = true;
        else a.bad = true;
    }
    ~Buffer()
    {
        if (held) PyBuffer_Release(&b);
    }
    template <typename T>
    const T *data() const { return static_cast<const T *>(b.buf); }
};

#define DOL_CALL(expr)                \
    if (a.bad) return nullptr;        \
    dol_status st;                    \
    Py_BEGIN_ALLOW_THREADS            \
    st = (expr);                      \
    Py_END_ALLOW_THREADS              \
    return done(st)

PyObject *apply2(PyObject *, PyObject *const *v, Py_ssize_t n)
{
    Args a(v, n, 6);
    auto *x = a.ptr<dol_dist>(0), *y = a.ptr<dol_dist>(1);
    auto *f = a.ptr<dol_fn_table>(2);
    auto *p = a.ptr<dol_prov>(3);
    auto *o = a.ptr<dol_dist>(4);
    void *s = a.stream(5);
    DOL_CALL(dol_apply2(x, y, f, p, o, s));
}

PyObject *backward(PyObject *, PyObject *const *v, Py_ssize_t n)
{
    Args a(v, n, 5);
    auto *r = a.ptr<dol_op_record>(0);
    auto *g = a.ptr<float>(1), *ga = a.ptr<float>(2), *gb = a.ptr<float>(3);
    void *s = a.stream(4);
    DOL_CALL(dol_backward(r, g, ga, gb, s));
}

PyObject *filter(PyObject *, PyObject *const *v, Py_ssize_t n)
{
    Args a(v, n, 5);
    auto *d = a.ptr<dol_dist>(0);
    Buffer pred(a, 1);
    auto *p = a.ptr<dol_prov>(2);
    auto *o = a.ptr<dol_dist>(3);
    void *s = a.stream(4);
    DOL_CALL(dol_filter(d, pred.data<uint8_t>(), p, o, s));
}

PyObject *union_(PyObject *, PyObject *const *v, Py_ssize_t n)
{
    Args a(v, n, 5);
    auto *x = a.ptr<dol_dist>(0), *y = a.ptr<dol_dist>(1);
    auto *p = a.ptr<dol_prov>(2);
    auto *o = a.ptr<dol_dist>(3);
    void *s = a.stream(4);
    DOL_CALL(dol_union(x, y, p, o, s));
}

PyObject *nll_grad(PyObject *, PyObject *const *v, Py_ssize_t n)
{
    Args a(v, n, 4);
    auto *d = a.ptr<dol_dist>(0);
    auto *t = a.ptr<int32_t>(1);
    auto *g = a.ptr<float>(2);
    void *s = a.stream(3);
    DOL_CALL(dol_nll_grad(d, t, g, s));
}

PyObject *dtkp_init(PyObject *, PyObject *const *v, Py_ssize_t n)
{
    Args a(v, n, 4);
    auto *d = a.ptr<dol_dist>(0);
    Buffer facts(a, 1);
    auto *p = a.ptr<dol_prov>(2);
    void *s = a.stream(3);
    DOL_CALL(dol_dtkp_init(d, facts.data<int32_t>(), p, s));
}

PyObject *dtkp_apply2_input(PyObject *, PyObject *const *v, Py_ssize_t n)
{
    Args a(v, n, 6);
    auto *x = a.ptr<dol_dist>(0);
    Buffer facts(a, 1);
    auto *f = a.ptr<dol_fn_table>(2);
    auto *p = a.ptr<dol_prov>(3);
    auto *o = a.ptr<dol_dist>(4);
    void *s = a.stream(5);
    DOL_CALL(dol_dtkp_apply2_input(x, facts.data<int32_t>(), f, p, o, s));
}

PyObject *dtkp_backward(PyObject *, PyObject *const *v, Py_ssize_t n)
{
    Args a(v, n, 6);
    auto *d = a.ptr<dol_dist>(0);
    auto *p = a.ptr<dol_prov>(1);
    auto *g = a.ptr<float>(2);
    const int64_t ld = a.num(3);
    auto *gf = a.ptr<float>(4);
    void *s = a.stream(5);
    DOL_CALL(dol_dtkp_backward(d, p, g, ld, gf, s));
}

PyObject *fold_apply2(PyObject *, PyObject *const *v, Py_ssize_t n)
{
    Args a(v, n, 2);
    auto *f = a.ptr<dol_fold>(0);
    void *s = a.stream(1);
    DOL_CALL(dol_fold_apply2(f, s));
}

PyObject *dtkp_fold_apply2(PyObject *, PyObject *const *v, Py_ssize_t n)
{
    Args a(v, n, 3);
    auto *f = a.ptr<dol_dtkp_fold>(0);
    auto *p = a.ptr<dol_prov>(1);
    void *s = a.stream(2);
    DOL_CALL(dol_dtkp_fold_apply2(f, p, s));
}

// setup(fail, current_device, current_raw_stream)
PyObject *setup(PyObject *, PyObject *const *v, Py_ssize_t n)
{
    Args a(v, n, 3);
    if (a.bad) return nullptr;
    PyObject **to[3] = {&g_fail, &g_device, &g_stream};
    for (int k = 0; k < 3; ++k) {
        Py_INCREF(v[k]);
        Py_XSETREF(*to[k], v[k]);
    }
    Py_RETURN_NONE;
}

#define DOL_FAST(f) reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr
PyMethodDef g_methods[] = {
    {"setup", DOL_FAST(setup)},
    {"apply2", DOL_FAST(apply2)},
    {"backward", DOL_FAST(backward)},
    {"filter", DOL_FAST(filter)},
    {"union", DOL_FAST(union_)},
    {"nll_grad", DOL_FAST(nll_grad)},
    {"dtkp_init", DOL_FAST(dtkp_init)},
    {"dtkp_apply2_input", DOL_FAST(dtkp_apply2_input)},
    {"dtkp_backward", DOL_FAST(dtkp_backward)},
    {"fold_apply2", DOL_FAST(fold_apply2)},
    {"dtkp_fold_apply2", DOL_FAST(dtkp_fold_apply2)},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&g_module); }
