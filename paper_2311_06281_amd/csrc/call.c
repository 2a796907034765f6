/* The two scan entry points as Python calls: arguments taken as they are and handed to the library.
 *
 * The smallest calls are bound by the host.  ctypes takes about 0.5 us to convert ten arguments and a Python frame
 * with the four data_ptr() calls another 0.5, beside 3.1 us for the launch itself; here it is 0.4 together. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

typedef int (*scan_fn)(const void *, const void *, const void *, void *, int64_t, int64_t, int64_t, int, uint32_t, void *);

static scan_fn entry[2]; /* heinsen_scan, heinsen_scan_static */
static PyObject *name_data_ptr, *name_cuda_stream;

/* What `x`, a Python integer, holds, reduced to 64 bits as ctypes does it.  0: it is no integer. */
static int integer(PyObject *x, uint64_t *v)
{
    if (!PyLong_Check(x)) return 0;
    *v = PyLong_AsUnsignedLongLongMask(x);
    return 1;
}

/* Address behind `x`: None, an integer, or what its method or attribute `name` gives.  0: none of these (an exception
 * is set unless there is merely no integer). */
static int address(PyObject *x, PyObject *name, int is_method, uint64_t *v)
{
    if (x == Py_None) {
        *v = 0;
        return 1;
    }
    if (PyLong_CheckExact(x)) return integer(x, v);
    PyObject *r = is_method ? PyObject_CallMethodNoArgs(x, name) : PyObject_GetAttr(x, name);
    if (r == NULL) return 0;
    const int ok = integer(r, v);
    Py_DECREF(r);
    return ok;
}

/* (a, b, x0, out, B, D, n, layout, flags, stream) -> status, or NotImplemented where some argument is of another kind
 * than these (the caller then converts them one by one, which also says what is wrong). */
static PyObject *call(int which, PyObject *const *args, Py_ssize_t nargs)
{
    uint64_t p[4], v[5], stream;
    if (nargs != 10 || entry[which] == NULL) Py_RETURN_NOTIMPLEMENTED;
    /* where the caller deals in addresses and handles, its numbers are looked at before any tensor is asked for its own */
    if (PyLong_CheckExact(args[0]) || PyLong_CheckExact(args[9]) || args[9] == Py_None)
        for (int i = 0; i < 5; ++i)
            if (!PyLong_Check(args[4 + i])) goto other;
    for (int i = 0; i < 4; ++i)
        if (!address(args[i], name_data_ptr, 1, &p[i])) goto other;
    for (int i = 0; i < 5; ++i)
        if (!integer(args[4 + i], &v[i])) goto other;
    if (!address(args[9], name_cuda_stream, 0, &stream)) goto other;
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = entry[which]((const void *)(uintptr_t)p[0], (const void *)(uintptr_t)p[1], (const void *)(uintptr_t)p[2], (void *)(uintptr_t)p[3],
                          (int64_t)v[0], (int64_t)v[1], (int64_t)v[2], (int)v[3], (uint32_t)v[4], (void *)(uintptr_t)stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
other:
    if (PyErr_Occurred()) {
        if (!PyErr_ExceptionMatches(PyExc_AttributeError) && !PyErr_ExceptionMatches(PyExc_TypeError)) return NULL;
        PyErr_Clear();
    }
    Py_RETURN_NOTIMPLEMENTED;
}

static PyObject *scan(PyObject *self, PyObject *const *args, Py_ssize_t nargs) { return call(0, args, nargs); }
static PyObject *scan_static(PyObject *self, PyObject *const *args, Py_ssize_t nargs) { return call(1, args, nargs); }

/* bind(address of heinsen_scan, address of heinsen_scan_static) */
static PyObject *bind(PyObject *self, PyObject *args)
{
    unsigned long long f, g;
    if (!PyArg_ParseTuple(args, "KK", &f, &g)) return NULL;
    entry[0] = (scan_fn)(uintptr_t)f;
    entry[1] = (scan_fn)(uintptr_t)g;
    Py_RETURN_NONE;
}

static PyMethodDef methods[] = {
    {"scan", (PyCFunction)(void (*)(void))scan, METH_FASTCALL, NULL},
    {"scan_static", (PyCFunction)(void (*)(void))scan_static, METH_FASTCALL, NULL},
    {"bind", bind, METH_VARARGS, NULL},
    {NULL, NULL, 0, NULL},
};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_call", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__call(void)
{
    name_data_ptr = PyUnicode_InternFromString("data_ptr");
    name_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    if (name_data_ptr == NULL || name_cuda_stream == NULL) return NULL;
    return PyModule_Create(&module);
}
