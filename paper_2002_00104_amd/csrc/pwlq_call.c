/* Calls of the library from Python without ctypes: _pwlq_call.search, .quantize and .linear_i8.
 *
 * A call of one small tensor is bound by the host: of 5.0 us for an inner product of 8 x 256 x 64, the launch
 * included, 0.9 us were ctypes converting sixteen arguments and 1.4 us the binding around it.
 * A function takes the address of the library's function (ctypes knows it), then that function's arguments;
 * where it has a pointer, a tensor (its data_ptr() is asked for here), an address, or None.  The
 * interpreter's lock is released during the call.  Returns the library's status. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

static PyObject *data_ptr_name;

static int64_t whole(PyObject *o, int *bad)
{
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) *bad = 1;
    return v;
}

static int small(PyObject *o, int *bad)
{
    const int64_t v = whole(o, bad);
    if (!*bad && v != (int)v) {
        PyErr_SetString(PyExc_OverflowError, "an argument does not fit an int");
        *bad = 1;
    }
    return (int)v;
}

static float real(PyObject *o, int *bad)
{
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) *bad = 1;
    return (float)v;
}

static void *pointer(PyObject *o, int *bad)
{
    void *p;
    if (*bad || o == Py_None) return NULL;
    if (PyLong_Check(o)) p = PyLong_AsVoidPtr(o);
    else {
        PyObject *v = PyObject_CallMethodNoArgs(o, data_ptr_name);
        if (!v) {
            *bad = 1;
            return NULL;
        }
        p = PyLong_AsVoidPtr(v);
        Py_DECREF(v);
    }
    if (!p && PyErr_Occurred()) *bad = 1;
    return p;
}

static int count(const char *name, Py_ssize_t got, Py_ssize_t want)
{
    if (got == want) return 1;
    PyErr_Format(PyExc_TypeError, "%s takes %zd arguments, %zd given", name, want, got);
    return 0;
}

#define PTR(i) pointer(a[i], &bad)
#define INT(i) small(a[i], &bad)
#define I64(i) whole(a[i], &bad)
#define F32(i) real(a[i], &bad)

typedef int (*SearchFn)(const void *, int64_t, int64_t, int, int, int, void *, void *, void *, void *, void *, size_t,
                        void *);

/* fn, w, C, K, bits, n_cand, mode, p_star, m, k_star, mse, workspace, workspace_bytes, stream */
static PyObject *call_search(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    int bad = 0, rc;
    (void)self;
    if (!count("search", n, 14)) return NULL;
    SearchFn fn = (SearchFn)PTR(0);
    void *w = PTR(1), *p = PTR(7), *m = PTR(8), *k = PTR(9), *mse = PTR(10), *ws = PTR(11), *stream = PTR(13);
    const int64_t C = I64(2), K = I64(3), bytes = I64(12);
    const int bits = INT(4), cand = INT(5), mode = INT(6);
    if (bad) return NULL;
    Py_BEGIN_ALLOW_THREADS
    rc = fn(w, C, K, bits, cand, mode, p, m, k, mse, ws, (size_t)bytes, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

typedef int (*QuantizeFn)(const void *, int64_t, int64_t, int, int, const void *, const void *, void *, void *, void *,
                          void *);

/* fn, w, C, K, bits, mode, p_star, m, codes, flags, w_hat, stream */
static PyObject *call_quantize(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    int bad = 0, rc;
    (void)self;
    if (!count("quantize", n, 12)) return NULL;
    QuantizeFn fn = (QuantizeFn)PTR(0);
    void *w = PTR(1), *p = PTR(6), *m = PTR(7), *codes = PTR(8), *flags = PTR(9), *hat = PTR(10), *stream = PTR(11);
    const int64_t C = I64(2), K = I64(3);
    const int bits = INT(4), mode = INT(5);
    if (bad) return NULL;
    Py_BEGIN_ALLOW_THREADS
    rc = fn(w, C, K, bits, mode, p, m, codes, flags, hat, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

typedef int (*LinearFn)(const void *, int64_t, int64_t, float, float, const void *, const void *, int64_t, int,
                        const void *, const void *, void *, void *, void *, size_t, void *);

/* fn, xq, M, K, s_x, z_x, packed_codes, packed_flags, N, bits, p, m, y, acc, workspace, workspace_bytes, stream */
static PyObject *call_linear(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    int bad = 0, rc;
    (void)self;
    if (!count("linear_i8", n, 17)) return NULL;
    LinearFn fn = (LinearFn)PTR(0);
    void *xq = PTR(1), *codes = PTR(6), *flags = PTR(7), *p = PTR(10), *m = PTR(11), *y = PTR(12), *acc = PTR(13),
         *ws = PTR(14), *stream = PTR(16);
    const int64_t M = I64(2), K = I64(3), N = I64(8), bytes = I64(15);
    const float s_x = F32(4), z_x = F32(5);
    const int bits = INT(9);
    if (bad) return NULL;
    Py_BEGIN_ALLOW_THREADS
    rc = fn(xq, M, K, s_x, z_x, codes, flags, N, bits, p, m, y, acc, ws, (size_t)bytes, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

static PyMethodDef methods[] = {
    {"search", (PyCFunction)(void (*)(void))call_search, METH_FASTCALL, NULL},
    {"quantize", (PyCFunction)(void (*)(void))call_quantize, METH_FASTCALL, NULL},
    {"linear_i8", (PyCFunction)(void (*)(void))call_linear, METH_FASTCALL, NULL},
    {NULL, NULL, 0, NULL}};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pwlq_call", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__pwlq_call(void)
{
    data_ptr_name = PyUnicode_InternFromString("data_ptr");
    return data_ptr_name ? PyModule_Create(&module) : NULL;
}
