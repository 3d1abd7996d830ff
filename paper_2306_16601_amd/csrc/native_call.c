/* CPython entry points spmm_run and spmm_run_tiled: argument marshalling of one launch, in C.
 *
 * A launch of the short-batch kernels lasts about 3 us and hipLaunchKernel about the same on the
 * host; marshalling the same eight arguments through ctypes and checking the extents of the two
 * tensors in Python took another 4 us per call, which made the interpreter the limit of every
 * short launch (768x768, 32 tokens, calls back to back: 7.2 us through ctypes, 4.5 us this way).
 *
 * The module holds no library of its own: binding.py hands over the addresses of the three C
 * functions once it has loaded the library (load(), called here on the first launch).
 */
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include "spmm.h"

typedef spmm_status_t (*run_fn)(const spmm_handle_t *, const uint8_t *, int64_t, int64_t, const spmm_epilogue_t *, void *,
                                int64_t, void *);
typedef spmm_status_t (*run_tiled_fn)(const spmm_handle_t *, const uint8_t *, int64_t, int64_t, const spmm_epilogue_t *,
                                      void *, int64_t, uint32_t, void *);
typedef spmm_status_t (*info_fn)(const spmm_handle_t *, int64_t *, int64_t *, int64_t *, int64_t *, int64_t *);

static run_fn p_run;
static run_tiled_fn p_run_tiled;
static info_fn p_info;
static PyObject *py_load, *py_check_extents, *py_check; /* binding.py: lib, _check_extents, _check */
static PyObject *s_data_ptr, *s_nbytes, *s_is_contiguous;

/* int(x) as a 64-bit value; -1 with an exception set on failure */
static int64_t as_i64(PyObject *x)
{
    if (PyLong_CheckExact(x)) return PyLong_AsLongLong(x);
    PyObject *v = PyNumber_Long(x);
    if (!v) return -1;
    const int64_t r = PyLong_AsLongLong(v);
    Py_DECREF(v);
    return r;
}

/* Address of an operand: a tensor's data_ptr(), a raw integer, or NULL for None. */
static int as_address(PyObject *x, void **out, int *is_tensor)
{
    *out = NULL;
    *is_tensor = 0;
    if (x == Py_None) return 0;
    PyObject *v = NULL;
    if (!PyLong_CheckExact(x)) {
        v = PyObject_CallMethodNoArgs(x, s_data_ptr);
        if (v) {
            *is_tensor = 1;
        } else {
            if (!PyErr_ExceptionMatches(PyExc_AttributeError)) return -1;
            PyErr_Clear();
            v = PyNumber_Long(x);
            if (!v) return -1;
        }
        x = v;
    }
    *out = (void *)(uintptr_t)PyLong_AsUnsignedLongLongMask(x);
    Py_XDECREF(v);
    return PyErr_Occurred() ? -1 : 0;
}

/* 1: the tensor is contiguous and holds at least `need` bytes, so the memory behind it does too.
 * 0: not known (the caller asks the exact check in binding.py). */
static int surely_covers(PyObject *t, __int128 need)
{
    int ok = 0;
    PyObject *c = PyObject_CallMethodNoArgs(t, s_is_contiguous), *n = NULL;
    if (c == Py_True && (n = PyObject_GetAttr(t, s_nbytes)) && PyLong_CheckExact(n)) {
        const long long have = PyLong_AsLongLong(n);
        ok = have >= 0 && (__int128)have >= need;
    }
    Py_XDECREF(c);
    Py_XDECREF(n);
    PyErr_Clear();
    return ok;
}

enum { A_HANDLE, A_X, A_M, A_LDX, A_EP, A_OUT, A_LDO, A_TILED, A_STREAM, A_COUNT };
static const char *const names[A_COUNT] = {"handle", "X_dev", "M", "ldx", "ep", "out_dev", "ldo", "tiled", "stream"};

static PyObject *launch(PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames, const int tiled_call)
{
    const char *const fname = tiled_call ? "spmm_run_tiled" : "spmm_run";
    /* positions of spmm_run skip A_TILED */
    PyObject *a[A_COUNT] = {0};
    const Py_ssize_t most = tiled_call ? A_COUNT : A_COUNT - 1;
    if (nargs > most) return PyErr_Format(PyExc_TypeError, "%s() takes at most %zd arguments (%zd given)", fname, most, nargs);
    for (Py_ssize_t i = 0; i < nargs; ++i) a[i + (!tiled_call && i >= A_TILED)] = args[i];
    for (Py_ssize_t k = 0; kwnames && k < PyTuple_GET_SIZE(kwnames); ++k) {
        PyObject *name = PyTuple_GET_ITEM(kwnames, k);
        int i = 0;
        while (i < A_COUNT && ((i == A_TILED && !tiled_call) || PyUnicode_CompareWithASCIIString(name, names[i]) != 0)) ++i;
        if (i == A_COUNT) return PyErr_Format(PyExc_TypeError, "%s() got an unexpected keyword argument '%U'", fname, name);
        if (a[i]) return PyErr_Format(PyExc_TypeError, "%s() got multiple values for argument '%s'", fname, names[i]);
        a[i] = args[nargs + k];
    }
    for (int i = 0; i < A_STREAM; ++i)
        if (!a[i] && !(i == A_TILED && !tiled_call))
            return PyErr_Format(PyExc_TypeError, "%s() missing required argument '%s'", fname, names[i]);

    if (!p_run) { /* first launch of the process: load the library, which binds this module */
        PyObject *r = PyObject_CallNoArgs(py_load);
        if (!r) return NULL;
        Py_DECREF(r);
        if (!p_run) return PyErr_Format(PyExc_RuntimeError, "the library did not bind its launch functions");
    }

    void *handle, *X, *out, *stream = NULL;
    int ignored, x_tensor, out_tensor;
    if (as_address(a[A_HANDLE], &handle, &ignored) < 0 || as_address(a[A_X], &X, &x_tensor) < 0 ||
        as_address(a[A_OUT], &out, &out_tensor) < 0)
        return NULL;
    if (a[A_STREAM] && as_address(a[A_STREAM], &stream, &ignored) < 0) return NULL;
    const int64_t M = as_i64(a[A_M]), ldx = as_i64(a[A_LDX]), ldo = as_i64(a[A_LDO]);
    const int64_t tiled = tiled_call ? as_i64(a[A_TILED]) : 0;
    if (PyErr_Occurred()) return NULL;

    Py_buffer epb = {0};
    const spmm_epilogue_t *ep = NULL;
    if (a[A_EP] != Py_None) {
        if (PyObject_GetBuffer(a[A_EP], &epb, PyBUF_SIMPLE) < 0) return NULL;
        if (epb.len != (Py_ssize_t)sizeof(spmm_epilogue_t)) {
            PyBuffer_Release(&epb);
            return PyErr_Format(PyExc_TypeError, "%s(): ep is not an spmm_epilogue_t", fname);
        }
        ep = (const spmm_epilogue_t *)epb.buf;
    }

    /* operands given as tensors must cover what the call touches (M <= 0 is rejected by the library) */
    if ((x_tensor || out_tensor) && M > 0) {
        int64_t N = 0, K = 0;
        int sure = p_info((const spmm_handle_t *)handle, &N, &K, NULL, NULL, NULL) == SPMM_OK;
        if (sure) {
            const __int128 tiles = (M + SPMM_X_TILE - 1) / SPMM_X_TILE;
            const int esz = ep && (ep->out_type == SPMM_OUT_S32 || ep->out_type == SPMM_OUT_F32) ? 4 : 1;
            const __int128 need_x = (tiled & SPMM_TILED_X) ? tiles * K * SPMM_X_TILE : (__int128)(K - 1) * ldx + M;
            const __int128 need_o = (tiled & SPMM_TILED_OUT) ? tiles * N * SPMM_X_TILE : ((__int128)(N - 1) * ldo + M) * esz;
            sure = (!x_tensor || surely_covers(a[A_X], need_x)) && (!out_tensor || surely_covers(a[A_OUT], need_o));
        }
        if (!sure) { /* a view, or too small: the exact check, which raises where the memory does not suffice */
            PyObject *t = PyLong_FromLongLong(tiled);
            PyObject *r = t ? PyObject_CallFunctionObjArgs(py_check_extents, a[A_HANDLE], a[A_X], a[A_M], a[A_LDX], a[A_EP],
                                                           a[A_OUT], a[A_LDO], t, NULL)
                            : NULL;
            Py_XDECREF(t);
            if (!r) {
                if (epb.obj) PyBuffer_Release(&epb);
                return NULL;
            }
            Py_DECREF(r);
        }
    }

    spmm_status_t st;
    Py_BEGIN_ALLOW_THREADS
    if (tiled_call)
        st = p_run_tiled((const spmm_handle_t *)handle, (const uint8_t *)X, M, ldx, ep, out, ldo, (uint32_t)tiled, stream);
    else
        st = p_run((const spmm_handle_t *)handle, (const uint8_t *)X, M, ldx, ep, out, ldo, stream);
    Py_END_ALLOW_THREADS
    if (epb.obj) PyBuffer_Release(&epb);
    if (st != SPMM_OK) return PyObject_CallFunction(py_check, "is", (int)st, fname); /* raises SpmmError */
    Py_RETURN_NONE;
}

static PyObject *native_run(PyObject *self, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames)
{
    (void)self;
    return launch(args, nargs, kwnames, 0);
}

static PyObject *native_run_tiled(PyObject *self, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames)
{
    (void)self;
    return launch(args, nargs, kwnames, 1);
}

/* hooks(lib, _check_extents, _check): the functions of binding.py this module calls back */
static PyObject *native_hooks(PyObject *self, PyObject *args)
{
    PyObject *l, *e, *c;
    (void)self;
    if (!PyArg_ParseTuple(args, "OOO", &l, &e, &c)) return NULL;
    Py_INCREF(l); Py_INCREF(e); Py_INCREF(c);
    Py_XSETREF(py_load, l);
    Py_XSETREF(py_check_extents, e);
    Py_XSETREF(py_check, c);
    Py_RETURN_NONE;
}

/* bind(address of spmm_run, of spmm_run_tiled, of spmm_info) */
static PyObject *native_bind(PyObject *self, PyObject *args)
{
    unsigned long long r, t, i;
    (void)self;
    if (!PyArg_ParseTuple(args, "KKK", &r, &t, &i)) return NULL;
    p_info = (info_fn)(uintptr_t)i;
    p_run_tiled = (run_tiled_fn)(uintptr_t)t;
    p_run = (run_fn)(uintptr_t)r;
    Py_RETURN_NONE;
}

static PyMethodDef methods[] = {
    {"spmm_run", (PyCFunction)(void (*)(void))native_run, METH_FASTCALL | METH_KEYWORDS,
     "spmm_run(handle, X_dev, M, ldx, ep, out_dev, ldo, stream=None)\n--\n\n"
     "out = postops(W . X), asynchronous on `stream` (a raw hipStream_t value, None = default stream)."},
    {"spmm_run_tiled", (PyCFunction)(void (*)(void))native_run_tiled, METH_FASTCALL | METH_KEYWORDS,
     "spmm_run_tiled(handle, X_dev, M, ldx, ep, out_dev, ldo, tiled, stream=None)\n--\n\n"
     "spmm_run with X (SPMM_TILED_X) and / or a 1-byte output (SPMM_TILED_OUT) in token-tile-major order."},
    {"hooks", native_hooks, METH_VARARGS, NULL},
    {"bind", native_bind, METH_VARARGS, NULL},
    {NULL, NULL, 0, NULL}};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native_call", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__native_call(void)
{
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_nbytes = PyUnicode_InternFromString("nbytes");
    s_is_contiguous = PyUnicode_InternFromString("is_contiguous");
    if (!s_data_ptr || !s_nbytes || !s_is_contiguous) return NULL;
    return PyModule_Create(&module);
}
