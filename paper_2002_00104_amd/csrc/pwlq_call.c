/* Calls of the library from Python without ctypes: _pwlq_call.search, .quantize and .linear_i8.
 *
 * A call of one small tensor is bound by the host: of 5.0 us for an inner product of 8 x 256 x 64, the launch
 * included, 0.9 us were ctypes converting sixteen arguments and 1.4 us the binding around it.
 * A function takes the address of the library's function (ctypes knows it), then that function's arguments;
 * where it has a pointer, a tensor (its data_ptr() is asked for here), or None where the library takes NULL.
 * An integer is taken for the function and for the stream only: in the place of a tensor it would reach a
 * kernel as a device address.  The interpreter's lock is released during the call.  Returns the library's status. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

static PyObject *data_ptr_name;

static int64_t whole(PyObject *o, int *bad)
{
    const long long v = *bad ? 0 : PyLong_AsLongLong(o);
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
    const double v = *bad ? 0.0 : PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) *bad = 1;
    return (float)v;
}

/* The function or the stream. */
static void *handle(PyObject *o, int *bad)
{
    void *p;
    if (*bad) return NULL;
    if (!PyLong_Check(o)) {
        PyErr_SetString(PyExc_TypeError, "the function and the stream are integers");
        *bad = 1;
        return NULL;
    }
    p = PyLong_AsVoidPtr(o);
    if (!p && PyErr_Occurred()) *bad = 1;
    return p;
}

static void *function(PyObject *o, int *bad)
{
    void *p = handle(o, bad);
    if (!p && !*bad) {
        PyErr_SetString(PyExc_TypeError, "the function is NULL");
        *bad = 1;
    }
    return p;
}

static void *tensor(PyObject *o, int *bad)
{
    PyObject *v = *bad ? NULL : PyObject_CallMethodNoArgs(o, data_ptr_name);
    void *p = NULL;
    if (v) {
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

#define FN(i) function(a[i], &bad)
#define TENSOR(i) tensor(a[i], &bad)
#define TENSOR_OR_NONE(i) (a[i] == Py_None ? NULL : tensor(a[i], &bad))
#define STREAM(i) handle(a[i], &bad)
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
    SearchFn fn = (SearchFn)FN(0);
    void *w = TENSOR(1), *p = TENSOR(7), *m = TENSOR(8), *k = TENSOR(9), *mse = TENSOR(10), *ws = TENSOR(11), *stream = STREAM(13);
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
    QuantizeFn fn = (QuantizeFn)FN(0);
    void *w = TENSOR(1), *p = TENSOR(6), *m = TENSOR(7), *codes = TENSOR(8), *flags = TENSOR(9), *hat = TENSOR_OR_NONE(10),
         *stream = STREAM(11);
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
    LinearFn fn = (LinearFn)FN(0);
    void *xq = TENSOR(1), *codes = TENSOR(6), *flags = TENSOR(7), *p = TENSOR(10), *m = TENSOR(11), *y = TENSOR(12), *acc = TENSOR_OR_NONE(13),
         *ws = TENSOR(14), *stream = STREAM(16);
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
