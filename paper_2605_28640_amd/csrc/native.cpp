// The per-token calls of the binding (append, decode, replayable step) with their arguments taken apart in C++: ctypes and a
// Python function per tensor cost the host more than the launch itself.  Same checks, same errors, same conversions;
// the library's functions come in as addresses (setup), so this module links against Python and torch only.
#define PY_SSIZE_T_CLEAN
#include <torch/csrc/autograd/python_variable.h>

#include <cstring>
#include <exception>

#include "../../include/ratsparse.h"

namespace {

decltype(&rat_scan) f_scan;
decltype(&sparse_attn_decode) f_decode;
decltype(&rat_decode_step) f_step;
PyObject *g_ptr, *g_check, *g_stream_of, *g_device, *g_workspace;  // binding._ptr, binding._check, torch's two, binding.Workspace
PyObject *s_buf, *s_ptr, *s_nbytes;

// One call's arguments.  Every getter leaves a Python exception and ok = false behind on failure.
struct Args {
    PyObject *const *a;
    bool ok = true;

    // a device tensor's address; None: null
    void *tensor(int i)
    {
        PyObject *o = a[i];
        if (!ok || o == Py_None) return nullptr;
        if (THPVariable_CheckExact(o)) {
            try {
                const at::Tensor &t = THPVariable_Unpack(o);
                if (t.is_cuda() && t.is_contiguous()) return t.data_ptr();
            } catch (const std::exception &e) {
                PyErr_SetString(PyExc_RuntimeError, e.what());
                ok = false;
                return nullptr;
            }
        }
        // anything else: the Python function decides (and raises what it always has)
        return address(PyObject_CallOneArg(g_ptr, o));
    }
    void *address(PyObject *r)  // steals r
    {
        if (!r) {
            ok = false;
            return nullptr;
        }
        void *p = nullptr;
        if (r != Py_None) {
            p = (void *)PyLong_AsUnsignedLongLongMask(r);
            if (PyErr_Occurred()) ok = false;
        }
        Py_DECREF(r);
        return p;
    }
    int64_t integer(int i)
    {
        if (!ok) return 0;
        const unsigned long long x = PyLong_AsUnsignedLongLongMask(a[i]);
        if (x == (unsigned long long)-1 && PyErr_Occurred()) ok = false;
        return (int64_t)x;
    }
    float real(int i)
    {
        if (!ok) return 0.f;
        const double x = PyFloat_AsDouble(a[i]);
        if (x == -1.0 && PyErr_Occurred()) ok = false;
        return (float)x;
    }
    // the shape structure (a ctypes one: it exports its memory)
    rs_shape shape(int i)
    {
        rs_shape s = {};
        Py_buffer b;
        if (!ok) return s;
        if (PyObject_GetBuffer(a[i], &b, PyBUF_SIMPLE) != 0) {
            ok = false;
            return s;
        }
        if (b.len == (Py_ssize_t)sizeof(s)) memcpy(&s, b.buf, sizeof(s));
        else {
            PyErr_SetString(PyExc_TypeError, "a shape from make_shape is expected");
            ok = false;
        }
        PyBuffer_Release(&b);
        return s;
    }
    // a workspace's buffer; a false value: none
    void *workspace(int i, size_t &bytes)
    {
        bytes = 0;
        PyObject *o = a[i];
        if (!ok || o == Py_None) return nullptr;
        if ((PyObject *)Py_TYPE(o) == g_workspace) {
            PyObject *buf = PyObject_GetAttr(o, s_buf);
            if (buf && THPVariable_CheckExact(buf)) {
                void *p = nullptr;
                try {
                    const at::Tensor &t = THPVariable_Unpack(buf);
                    p = t.data_ptr();
                    bytes = (size_t)t.numel();
                } catch (const std::exception &e) {
                    PyErr_SetString(PyExc_RuntimeError, e.what());
                    ok = false;
                }
                Py_DECREF(buf);
                return p;
            }
            Py_XDECREF(buf);
            PyErr_Clear();
        }
        const int some = PyObject_IsTrue(o);
        if (some <= 0) {
            if (some < 0) ok = false;
            return nullptr;
        }
        void *p = address(PyObject_GetAttr(o, s_ptr));
        if (ok) bytes = (size_t)(uintptr_t)address(PyObject_GetAttr(o, s_nbytes));
        return p;
    }
};

// the current stream of the current device
void *stream(bool &ok)
{
    if (!ok) return nullptr;
    PyObject *dev = PyObject_CallNoArgs(g_device);
    PyObject *r = dev ? PyObject_CallOneArg(g_stream_of, dev) : nullptr;
    Py_XDECREF(dev);
    if (!r) {
        ok = false;
        return nullptr;
    }
    void *s = (void *)PyLong_AsUnsignedLongLongMask(r);
    Py_DECREF(r);
    if (PyErr_Occurred()) ok = false;
    return s;
}

PyObject *done(int status)
{
    if (status == 0) Py_RETURN_NONE;
    PyObject *code = PyLong_FromLong(status);
    PyObject *r = code ? PyObject_CallOneArg(g_check, code) : nullptr;  // raises
    Py_XDECREF(code);
    return r;
}

bool expect(Py_ssize_t n, Py_ssize_t want)
{
    if (n == want) return true;
    PyErr_Format(PyExc_TypeError, "%zd arguments expected, %zd given", want, n);
    return false;
}

PyObject *py_rat_scan(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (!expect(n, 12)) return nullptr;
    Args x{a};
    const rs_shape s = x.shape(0);
    void *k = x.tensor(1), *v = x.tensor(2), *g = x.tensor(3), *sk = x.tensor(4), *sv = x.tensor(5), *kc = x.tensor(6),
         *vc = x.tensor(7), *meta = x.tensor(11);
    const int64_t t0 = x.integer(8), T = x.integer(9);
    size_t nb;
    void *ws = x.workspace(10, nb), *st = stream(x.ok);
    if (!x.ok) return nullptr;
    int r;
    Py_BEGIN_ALLOW_THREADS
    r = f_scan(&s, k, v, (const float *)g, (float *)sk, (float *)sv, kc, vc, meta, t0, T, ws, nb, st);
    Py_END_ALLOW_THREADS
    return done(r);
}

PyObject *py_sparse_attn_decode(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (!expect(n, 15)) return nullptr;
    Args x{a};
    const rs_shape s = x.shape(0);
    void *q = x.tensor(1), *kc = x.tensor(2), *vc = x.tensor(3), *idx = x.tensor(6), *meta = x.tensor(8), *out = x.tensor(11),
         *lse = x.tensor(12), *idx_out = x.tensor(13);
    const int64_t T = x.integer(4);
    const float scale = x.real(5);
    const int K = (int)x.integer(7), n_first = (int)x.integer(9), n_local = (int)x.integer(10);
    size_t nb;
    void *ws = x.workspace(14, nb), *st = stream(x.ok);
    if (!x.ok) return nullptr;
    int r;
    Py_BEGIN_ALLOW_THREADS
    r = f_decode(&s, q, kc, vc, T, scale, (const int32_t *)idx, K, meta, n_first, n_local, out, (float *)lse, (int32_t *)idx_out, ws, nb, st);
    Py_END_ALLOW_THREADS
    return done(r);
}

PyObject *py_rat_decode_step(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (!expect(n, 19)) return nullptr;
    Args x{a};
    const rs_shape s = x.shape(0);
    void *k = x.tensor(1), *v = x.tensor(2), *g = x.tensor(3), *sk = x.tensor(4), *sv = x.tensor(5), *kc = x.tensor(6),
         *vc = x.tensor(7), *meta = x.tensor(8), *q = x.tensor(9), *out = x.tensor(15), *lse = x.tensor(16), *idx_out = x.tensor(17);
    const float scale = x.real(10);
    const int K = (int)x.integer(11), n_first = (int)x.integer(12), n_local = (int)x.integer(13);
    const int64_t T_max = x.integer(14);
    size_t nb;
    void *ws = x.workspace(18, nb), *st = stream(x.ok);
    if (!x.ok) return nullptr;
    int r;
    Py_BEGIN_ALLOW_THREADS
    r = f_step(&s, k, v, (const float *)g, (float *)sk, (float *)sv, kc, vc, meta, q, scale, K, n_first, n_local, T_max, out, (float *)lse,
               (int32_t *)idx_out, ws, nb, st);
    Py_END_ALLOW_THREADS
    return done(r);
}

// setup(address of rat_scan, of sparse_attn_decode, of rat_decode_step, _ptr, _check, stream of a device, current device, Workspace)
PyObject *py_setup(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (!expect(n, 8)) return nullptr;
    Args x{a};
    f_scan = (decltype(f_scan))x.integer(0);
    f_decode = (decltype(f_decode))x.integer(1);
    f_step = (decltype(f_step))x.integer(2);
    if (!x.ok) return nullptr;
    PyObject **keep[5] = {&g_ptr, &g_check, &g_stream_of, &g_device, &g_workspace};
    for (int i = 0; i < 5; ++i) {
        Py_INCREF(a[3 + i]);
        Py_XDECREF(*keep[i]);
        *keep[i] = a[3 + i];
    }
    Py_RETURN_NONE;
}

#define FAST(f) (PyCFunction)(void (*)(void))f, METH_FASTCALL, nullptr
PyMethodDef methods[] = {{"setup", FAST(py_setup)},
                         {"rat_scan", FAST(py_rat_scan)},
                         {"sparse_attn_decode", FAST(py_sparse_attn_decode)},
                         {"rat_decode_step", FAST(py_rat_decode_step)},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native()
{
    s_buf = PyUnicode_InternFromString("buf");
    s_ptr = PyUnicode_InternFromString("ptr");
    s_nbytes = PyUnicode_InternFromString("nbytes");
    return PyModule_Create(&module);
}
