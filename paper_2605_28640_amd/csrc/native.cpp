// The per-token calls of the binding (append, decode, replayable step) with their arguments taken apart in C++: ctypes and a
// Python function per tensor cost the host more than the launch itself.  Only arguments of exactly the types that a program
// ordinarily passes are taken here: rs_shape, contiguous device tensors (torch.Tensor or Parameter) or None, int, float, Workspace.
// Anything else leaves the call unmade and the function answers False: binding.py then makes it through ctypes, which
// accepts, converts or refuses the argument as for every other function of the library.
// The library's functions come in as addresses (setup), so this module links against Python and torch only.
#define PY_SSIZE_T_CLEAN
#include <torch/csrc/autograd/python_variable.h>

#include <cstring>
#include <exception>

#include "../../include/ratsparse.h"

namespace {

decltype(&rat_scan) f_scan;
decltype(&sparse_attn_decode) f_decode;
decltype(&rat_decode_step) f_step;
PyObject *g_check, *g_stream_of, *g_device, *g_shape, *g_workspace;  // binding._check, torch's two, binding.rs_shape, .Workspace
PyObject *s_buf;

// One call's arguments.  A getter that meets something else than its plain type clears `plain` and raises nothing.
struct Args {
    PyObject *const *a;
    bool plain = true;

    void *refuse()
    {
        plain = false;
        return nullptr;
    }
    // a device tensor's address; None: null
    void *tensor(int i)
    {
        PyObject *o = a[i];
        if (o == Py_None) return nullptr;
        if (!THPVariable_CheckExact(o)) return refuse();
        try {
            const at::Tensor &t = THPVariable_Unpack(o);
            return t.is_cuda() && t.is_contiguous() ? t.data_ptr() : refuse();
        } catch (const std::exception &) {
            return refuse();
        }
    }
    // the low bits of an int, as ctypes takes them
    int64_t integer(int i)
    {
        if (PyLong_Check(a[i])) return (int64_t)PyLong_AsUnsignedLongLongMask(a[i]);
        refuse();
        return 0;
    }
    float real(int i)
    {
        if (PyFloat_Check(a[i])) return (float)PyFloat_AS_DOUBLE(a[i]);
        refuse();
        return 0.f;
    }
    // the shape structure (a ctypes one: it exports its memory)
    rs_shape shape(int i)
    {
        rs_shape s = {};
        Py_buffer b;
        if ((PyObject *)Py_TYPE(a[i]) != g_shape) {
            refuse();
        } else if (PyObject_GetBuffer(a[i], &b, PyBUF_SIMPLE) != 0) {
            PyErr_Clear();
            refuse();
        } else {
            if (b.len == (Py_ssize_t)sizeof(s)) memcpy(&s, b.buf, sizeof(s));
            else refuse();
            PyBuffer_Release(&b);
        }
        return s;
    }
    // a workspace's buffer
    void *workspace(int i, size_t &bytes)
    {
        bytes = 0;
        if ((PyObject *)Py_TYPE(a[i]) != g_workspace) return refuse();
        PyObject *buf = PyObject_GetAttr(a[i], s_buf);
        void *p = nullptr;
        if (buf && THPVariable_CheckExact(buf)) {
            try {
                const at::Tensor &t = THPVariable_Unpack(buf);
                p = t.data_ptr();
                bytes = (size_t)t.numel();
            } catch (const std::exception &) {
                refuse();
            }
        } else {
            PyErr_Clear();
            refuse();
        }
        Py_XDECREF(buf);
        return p;
    }
};

// the current stream of the current device; false: a Python exception
bool stream(void *&s)
{
    PyObject *dev = PyObject_CallNoArgs(g_device);
    PyObject *r = dev ? PyObject_CallOneArg(g_stream_of, dev) : nullptr;
    Py_XDECREF(dev);
    if (!r) return false;
    s = (void *)PyLong_AsUnsignedLongLongMask(r);
    Py_DECREF(r);
    return !PyErr_Occurred();
}

// True; or the exception that binding._check raises for a status
PyObject *done(int status)
{
    if (status != 0) {
        PyObject *code = PyLong_FromLong(status);
        PyObject *r = code ? PyObject_CallOneArg(g_check, code) : nullptr;
        Py_XDECREF(code);
        if (!r) return nullptr;
        Py_DECREF(r);
    }
    Py_RETURN_TRUE;
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
    size_t nb = 0;
    void *ws = a[10] == Py_None ? nullptr : x.workspace(10, nb), *st = nullptr;  // (a run may do without)
    if (!x.plain) Py_RETURN_FALSE;
    if (!stream(st)) return nullptr;
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
    size_t nb = 0;
    void *ws = x.workspace(14, nb), *st = nullptr;
    if (!x.plain) Py_RETURN_FALSE;
    if (!stream(st)) return nullptr;
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
    size_t nb = 0;
    void *ws = x.workspace(18, nb), *st = nullptr;
    if (!x.plain) Py_RETURN_FALSE;
    if (!stream(st)) return nullptr;
    int r;
    Py_BEGIN_ALLOW_THREADS
    r = f_step(&s, k, v, (const float *)g, (float *)sk, (float *)sv, kc, vc, meta, q, scale, K, n_first, n_local, T_max, out, (float *)lse,
               (int32_t *)idx_out, ws, nb, st);
    Py_END_ALLOW_THREADS
    return done(r);
}

// setup(address of rat_scan, of sparse_attn_decode, of rat_decode_step, _check, stream of a device, current device,
// rs_shape, Workspace)
PyObject *py_setup(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (!expect(n, 8)) return nullptr;
    Args x{a};
    f_scan = (decltype(f_scan))x.integer(0);
    f_decode = (decltype(f_decode))x.integer(1);
    f_step = (decltype(f_step))x.integer(2);
    if (!x.plain) {
        PyErr_SetString(PyExc_TypeError, "setup: three addresses expected");
        return nullptr;
    }
    PyObject **keep[5] = {&g_check, &g_stream_of, &g_device, &g_shape, &g_workspace};
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
    return PyModule_Create(&module);
}
