/* The attention entry points of include/climber.h as Python calls, for callers whose calls are short: converts what a call passes
 * (tensors, device pointers, None; numbers; ctypes structures) in C.  By ctypes the conversions took 1.6 of a call's 4.9 us on the
 * host (4.9 -> 3.6), and two fp32 calls of one small user 10.5 us as a pass for 8.3 in their kernels, 8.7 this way.
 *
 * A function returns the entry point's code, or None where an argument is none of these: climber.py then takes ctypes' way,
 * which converts it or refuses it.  Nothing is kept from one call for the next. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

#include "../../include/climber.h"

static __typeof__(&climber_attn_history) attn_history_fn;
static __typeof__(&climber_attn_sumi) attn_sumi_fn;
static __typeof__(&climber_attn_history_bias) attn_history_bias_fn;
static __typeof__(&climber_attn_sumi_bias) attn_sumi_bias_fn;
static PyObject *config_type, *bias_type, *current_device, *raw_stream, *s_data_ptr, *s_cuda_stream;

static int unsigned_of(PyObject *o, void **p) /* takes the reference */
{
    if (!o) return 0;
    const int ok = PyLong_Check(o);
    if (ok) *p = (void *)(uintptr_t)PyLong_AsUnsignedLongLong(o);
    Py_DECREF(o);
    return ok && !PyErr_Occurred();
}

static int pointer(PyObject *o, void **p)
{
    if (o == Py_None) return *p = NULL, 1;
    if (PyLong_Check(o)) return unsigned_of(Py_NewRef(o), p);
    return unsigned_of(PyObject_CallMethodNoArgs(o, s_data_ptr), p);
}

static int stream_of(PyObject *o, void **p)
{
    if (o == Py_None) { /* torch's current one */
        PyObject *dev = PyObject_CallNoArgs(current_device);
        PyObject *s = dev ? PyObject_CallOneArg(raw_stream, dev) : NULL;
        Py_XDECREF(dev);
        return unsigned_of(s, p);
    }
    if (PyLong_Check(o)) return unsigned_of(Py_NewRef(o), p);
    return unsigned_of(PyObject_GetAttr(o, s_cuda_stream), p);
}

static int number(PyObject *o, int32_t *v)
{
    if (!PyLong_Check(o)) return 0;
    int over;
    const long x = PyLong_AsLongAndOverflow(o, &over);
    *v = (int32_t)x;
    return !over && x == *v;
}

static int structure(PyObject *o, PyObject *type, size_t bytes, Py_buffer *b)
{
    if (!PyObject_TypeCheck(o, (PyTypeObject *)type)) return 0;
    if (PyObject_GetBuffer(o, b, PyBUF_SIMPLE)) return 0;
    if ((size_t)b->len == bytes) return 1;
    PyBuffer_Release(b);
    return 0;
}

static PyObject *elsewhere(void)
{
    PyErr_Clear();
    Py_RETURN_NONE;
}

/* cfg, tau, q, k, v, scen, beh, cache, layer, o[, bias], stream */
static PyObject *history(PyObject *const *a, Py_ssize_t n, int with_bias)
{
    if (n != 11 + with_bias) return elsewhere();
    void *p[8], *o, *s;
    int32_t layer;
    Py_buffer cfg, bias;
    for (int i = 1; i < 8; ++i)
        if (!pointer(a[i], &p[i])) return elsewhere();
    if (!number(a[8], &layer) || !pointer(a[9], &o) || !stream_of(a[n - 1], &s)) return elsewhere();
    if (!structure(a[0], config_type, sizeof(climber_config), &cfg)) return elsewhere();
    if (with_bias && !structure(a[10], bias_type, sizeof(climber_rel_bias), &bias)) return PyBuffer_Release(&cfg), elsewhere();
    int code;
    Py_BEGIN_ALLOW_THREADS
    if (with_bias) code = attn_history_bias_fn(cfg.buf, p[1], p[2], p[3], p[4], p[5], p[6], p[7], layer, o, bias.buf, s);
    else code = attn_history_fn(cfg.buf, p[1], p[2], p[3], p[4], p[5], p[6], p[7], layer, o, s);
    Py_END_ALLOW_THREADS
    PyBuffer_Release(&cfg);
    if (with_bias) PyBuffer_Release(&bias);
    return PyLong_FromLong(code);
}

/* cfg, tau, cache, layer, q, k, v, cand_off, m_total, m_max, scen, beh, o[, bias], stream */
static PyObject *sumi(PyObject *const *a, Py_ssize_t n, int with_bias)
{
    if (n != 14 + with_bias) return elsewhere();
    void *p[13], *s;
    int32_t layer, m_total, m_max;
    Py_buffer cfg, bias;
    for (int i = 1; i < 13; ++i)
        if (i != 3 && i != 8 && i != 9 && !pointer(a[i], &p[i])) return elsewhere();
    if (!number(a[3], &layer) || !number(a[8], &m_total) || !number(a[9], &m_max) || !stream_of(a[n - 1], &s)) return elsewhere();
    if (!structure(a[0], config_type, sizeof(climber_config), &cfg)) return elsewhere();
    if (with_bias && !structure(a[13], bias_type, sizeof(climber_rel_bias), &bias)) return PyBuffer_Release(&cfg), elsewhere();
    int code;
    Py_BEGIN_ALLOW_THREADS
    if (with_bias) code = attn_sumi_bias_fn(cfg.buf, p[1], p[2], layer, p[4], p[5], p[6], p[7], m_total, m_max, p[10], p[11], p[12], bias.buf, s);
    else code = attn_sumi_fn(cfg.buf, p[1], p[2], layer, p[4], p[5], p[6], p[7], m_total, m_max, p[10], p[11], p[12], s);
    Py_END_ALLOW_THREADS
    PyBuffer_Release(&cfg);
    if (with_bias) PyBuffer_Release(&bias);
    return PyLong_FromLong(code);
}

static PyObject *attn_history(PyObject *m, PyObject *const *a, Py_ssize_t n) { return history(a, n, 0); }
static PyObject *attn_history_bias(PyObject *m, PyObject *const *a, Py_ssize_t n) { return history(a, n, 1); }
static PyObject *attn_sumi(PyObject *m, PyObject *const *a, Py_ssize_t n) { return sumi(a, n, 0); }
static PyObject *attn_sumi_bias(PyObject *m, PyObject *const *a, Py_ssize_t n) { return sumi(a, n, 1); }

/* bind(addresses of the four entry points, Config, RelBias, torch.cuda.current_device, torch's raw current stream) */
static PyObject *bind(PyObject *m, PyObject *args)
{
    unsigned long long f[4];
    PyObject *t[4];
    if (!PyArg_ParseTuple(args, "KKKKO!O!OO", &f[0], &f[1], &f[2], &f[3], &PyType_Type, &t[0], &PyType_Type, &t[1], &t[2], &t[3])) return NULL;
    attn_history_fn = (__typeof__(attn_history_fn))(uintptr_t)f[0];
    attn_sumi_fn = (__typeof__(attn_sumi_fn))(uintptr_t)f[1];
    attn_history_bias_fn = (__typeof__(attn_history_bias_fn))(uintptr_t)f[2];
    attn_sumi_bias_fn = (__typeof__(attn_sumi_bias_fn))(uintptr_t)f[3];
    PyObject **const to[4] = {&config_type, &bias_type, &current_device, &raw_stream};
    for (int i = 0; i < 4; ++i) {
        PyObject *was = *to[i];
        *to[i] = Py_NewRef(t[i]);
        Py_XDECREF(was);
    }
    Py_RETURN_NONE;
}

static PyMethodDef methods[] = {
    {"bind", bind, METH_VARARGS, NULL},
    {"attn_history", (PyCFunction)(void (*)(void))attn_history, METH_FASTCALL, NULL},
    {"attn_history_bias", (PyCFunction)(void (*)(void))attn_history_bias, METH_FASTCALL, NULL},
    {"attn_sumi", (PyCFunction)(void (*)(void))attn_sumi, METH_FASTCALL, NULL},
    {"attn_sumi_bias", (PyCFunction)(void (*)(void))attn_sumi_bias, METH_FASTCALL, NULL},
    {NULL, NULL, 0, NULL}};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__native(void)
{
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    return s_data_ptr && s_cuda_stream ? PyModule_Create(&module) : NULL;
}
