// The way from Python to a launch for the calls that decode and short prompts make by the dozen: what
// binding.py does for them in Python and ctypes, in C.  A call passes the same checks on the same methods
// of its tensors (shape, stride, data_ptr, is_contiguous), reads the stream through the same functions of
// torch and releases the interpreter lock while the library runs.  Anything out of the ordinary -- a
// method that raises an error, a number that is not a plain int or float, a layout the checks refuse --
// returns NotImplemented before the library is called, and binding.py goes its own way, which also
// words the errors.  Nothing is kept from one call for another.
//
// A call through this file costs the host 1.0 us beside the launch, through ctypes 3.3 (512 -> 512 at T = 64, a 3.8 us
// kernel: 6.0 -> 4.0, 6.4 -> 5.0 and 6.8 -> 4.9 us a call on three machines).
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <stdint.h>

#include "mquant.h"

static PyObject *s_shape, *s_stride, *s_data_ptr, *s_is_contiguous;

// What setup() gives a module object: torch.cuda.is_initialized, the current device, its raw stream, and the library's
// entries.  Every load of the package has a module, and so a library, of its own.
typedef struct {
    PyObject *f_initialized, *f_device, *f_stream;
    int (*prefill)(const void *, int64_t, const int32_t *, const uint8_t *, const void *, void *, int64_t, int32_t, int32_t,
                   int32_t, int32_t, float, float, int32_t, void *, int64_t, mquant_stream_t);
    int (*prefill_static)(const void *, int64_t, const int32_t *, const uint8_t *, const void *, void *, int64_t, int32_t,
                          int32_t, int32_t, int32_t, float, float, int32_t, mquant_stream_t);
    int (*decode)(const void *, int64_t, const uint8_t *, const void *, void *, int64_t, int32_t, int32_t, int32_t, int32_t,
                  float, float, int32_t, mquant_stream_t);
    int (*decode_grouped)(const void *, int64_t, int32_t, int32_t, int32_t, float, float, int32_t, const mquant_linear_t *,
                          int32_t, mquant_stream_t);
    int (*gemv_grouped)(const int8_t *, int32_t, int32_t, int32_t, float, float, const mquant_linear_t *, int32_t,
                        mquant_stream_t);
    int (*quant)(const void *, int64_t, const int32_t *, int8_t *, int32_t, int32_t, int32_t, float, float, int32_t,
                 mquant_stream_t);
    int (*weight_only)(const void *, int64_t, const uint8_t *, void *, int64_t, int32_t, int32_t, int32_t, mquant_stream_t);
} State;

// ---- readers: 1 on success, 0 where the slow way has to look.  An interrupt, an exit and exhausted memory are nobody's
// layout: they stay set, and the call raises them.
static int no(void)
{
    if (PyErr_ExceptionMatches(PyExc_Exception) && !PyErr_ExceptionMatches(PyExc_MemoryError)) PyErr_Clear();
    return 0;
}

static int read_i64(PyObject *o, int64_t *v)
{
    if (!o || !PyLong_CheckExact(o)) return 0;
    *v = PyLong_AsLongLong(o);
    return *v != -1 || !PyErr_Occurred() ? 1 : no();
}

static int read_i32(PyObject *o, int32_t *v)
{
    int64_t w;
    if (!read_i64(o, &w) || w < INT32_MIN || w > INT32_MAX) return 0;
    *v = (int32_t)w;
    return 1;
}

static int read_f32(PyObject *o, float *v)
{
    if (!PyFloat_CheckExact(o)) return 0;
    *v = (float)PyFloat_AS_DOUBLE(o);
    return 1;
}

static int read_ptr(PyObject *t, void **p)                  // None: NULL
{
    *p = NULL;
    if (t == Py_None) return 1;
    PyObject *r = PyObject_VectorcallMethod(s_data_ptr, &t, 1 | PY_VECTORCALL_ARGUMENTS_OFFSET, NULL);
    if (!r) return no();
    if (PyLong_CheckExact(r)) *p = PyLong_AsVoidPtr(r);
    const int ok = PyLong_CheckExact(r) && !PyErr_Occurred();
    Py_DECREF(r);
    return ok ? 1 : no();
}

static int read_pair(PyObject *t, int64_t *a, int64_t *b)   // steals t
{
    if (!t) return no();
    const int ok = PyTuple_Check(t) && PyTuple_GET_SIZE(t) == 2 && read_i64(PyTuple_GET_ITEM(t, 0), a) &&
                   read_i64(PyTuple_GET_ITEM(t, 1), b);
    Py_DECREF(t);
    return ok;
}

// A 2-D operand with a leading dimension: unit stride along a row.
static int read_rows(PyObject *t, void **p, int64_t *ld, int64_t *rows, int64_t *cols)
{
    int64_t unit;
    if (t == Py_None || !read_pair(PyObject_GetAttr(t, s_shape), rows, cols)) return 0;
    if (!read_pair(PyObject_VectorcallMethod(s_stride, &t, 1 | PY_VECTORCALL_ARGUMENTS_OFFSET, NULL), ld, &unit)) return 0;
    if ((unit != 1 && *cols > 1) || (*ld < *cols && *rows > 1)) return 0;
    return read_ptr(t, p);
}

static int read_dense(PyObject *t, void **p)
{
    if (t != Py_None) {
        PyObject *r = PyObject_VectorcallMethod(s_is_contiguous, &t, 1 | PY_VECTORCALL_ARGUMENTS_OFFSET, NULL);
        if (!r) return no();
        const int ok = r == Py_True;
        Py_DECREF(r);
        if (!ok) return 0;
    }
    return read_ptr(t, p);
}

static int read_stream(const State *m, mquant_stream_t *s)
{
    if (!m->f_stream) return 0;
    PyObject *r = PyObject_CallNoArgs(m->f_initialized);
    if (!r) return no();
    const int up = r == Py_True;
    Py_DECREF(r);
    if (!up || !(r = PyObject_CallNoArgs(m->f_device))) return no();
    PyObject *st = PyObject_CallOneArg(m->f_stream, r);
    Py_DECREF(r);
    if (!st) return no();
    int ok = PyLong_CheckExact(st);
    if (ok) *s = PyLong_AsVoidPtr(st);
    ok = ok && !PyErr_Occurred();
    Py_DECREF(st);
    return ok ? 1 : no();
}

static int read_size(int64_t v, int32_t *out)
{
    *out = (int32_t)v;
    return v >= 0 && v <= INT32_MAX;
}

// (w_prepacked, w_scale, N, out) tuples
static int read_linears(PyObject *list, mquant_linear_t *lin, int32_t *n)
{
    if (!PyList_CheckExact(list) && !PyTuple_CheckExact(list)) return 0;
    const Py_ssize_t len = PySequence_Fast_GET_SIZE(list);
    if (len < 1 || len > 4) return 0;
    for (Py_ssize_t i = 0; i < len; ++i) {
        // a method called below may change the list
        if (PySequence_Fast_GET_SIZE(list) != len) return 0;
        PyObject *t = PySequence_Fast_GET_ITEM(list, i);
        if (!PyTuple_CheckExact(t) || PyTuple_GET_SIZE(t) != 4) return 0;
        Py_INCREF(t);
        void *w, *s, *y;
        int64_t rows, cols;
        const int ok = read_i32(PyTuple_GET_ITEM(t, 2), &lin[i].N) &&
                       read_rows(PyTuple_GET_ITEM(t, 3), &y, &lin[i].ldy, &rows, &cols) &&
                       read_dense(PyTuple_GET_ITEM(t, 1), &s) && read_ptr(PyTuple_GET_ITEM(t, 0), &w);
        Py_DECREF(t);
        if (!ok) return 0;
        lin[i].w_prepacked_dev = w;
        lin[i].w_scale_dev = s;
        lin[i].y_dev = y;
    }
    *n = (int32_t)len;
    return 1;
}

#define SLOW_WAY return slow_way()
static PyObject *slow_way(void)
{
    if (PyErr_Occurred()) return NULL;
    Py_RETURN_NOTIMPLEMENTED;
}

#define LAUNCH(...)                     \
    int st;                             \
    Py_BEGIN_ALLOW_THREADS              \
    st = __VA_ARGS__;                   \
    Py_END_ALLOW_THREADS                \
    return PyLong_FromLong(st)

// ---- entries: the arguments of the functions of binding.py, in order, all positional
static PyObject *prefill_any(const State *m, PyObject *const *a, Py_ssize_t n, int on_scratch)
{
    // x, perm, w_prepacked, w_scale, N, n_vis, s_vis, s_txt, had_block, out [, workspace, its bytes]
    void *x, *perm, *w, *ws, *y, *work = NULL;
    int64_t ldx, ldy, T, K, r, c, bytes = 0;
    int32_t T32, K32, N, n_vis, block;
    float s_vis, s_txt;
    mquant_stream_t s;
    if (n != (on_scratch ? 10 : 12) || !read_rows(a[0], &x, &ldx, &T, &K) || !read_rows(a[9], &y, &ldy, &r, &c) ||
        !read_size(T, &T32) || !read_size(K, &K32) || !read_dense(a[1], &perm) || !read_dense(a[3], &ws) ||
        !read_ptr(a[2], &w) || !read_i32(a[4], &N) || !read_i32(a[5], &n_vis) || !read_f32(a[6], &s_vis) ||
        !read_f32(a[7], &s_txt) || !read_i32(a[8], &block))
        SLOW_WAY;
    if (!on_scratch && (!read_ptr(a[10], &work) || !read_i64(a[11], &bytes))) SLOW_WAY;
    if (!read_stream(m, &s)) SLOW_WAY;
    if (on_scratch) {
        LAUNCH(m->prefill_static(x, ldx, perm, w, ws, y, ldy, T32, N, K32, n_vis, s_vis, s_txt, block, s));
    }
    LAUNCH(m->prefill(x, ldx, perm, w, ws, y, ldy, T32, N, K32, n_vis, s_vis, s_txt, block, work, bytes, s));
}

static PyObject *prefill(PyObject *self, PyObject *const *a, Py_ssize_t n) { return prefill_any(PyModule_GetState(self), a, n, 0); }
static PyObject *prefill_static(PyObject *self, PyObject *const *a, Py_ssize_t n) { return prefill_any(PyModule_GetState(self), a, n, 1); }

static PyObject *decode_grouped(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    const State *m = PyModule_GetState(self);
    // x, linears, n_vis, s_vis, s_txt, had_block
    void *x;
    int64_t ldx, T, K;
    int32_t T32, K32, n_vis, block, count;
    float s_vis, s_txt;
    mquant_linear_t lin[4];
    mquant_stream_t s;
    if (n != 6 || !read_rows(a[0], &x, &ldx, &T, &K) || !read_size(T, &T32) || !read_size(K, &K32) ||
        !read_linears(a[1], lin, &count) || !read_i32(a[2], &n_vis) || !read_f32(a[3], &s_vis) ||
        !read_f32(a[4], &s_txt) || !read_i32(a[5], &block) || !read_stream(m, &s))
        SLOW_WAY;
    LAUNCH(m->decode_grouped(x, ldx, T32, K32, n_vis, s_vis, s_txt, block, lin, count, s));
}

static PyObject *decode(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    const State *m = PyModule_GetState(self);
    // x, w_prepacked, w_scale, N, n_vis, s_vis, s_txt, had_block, out
    void *x, *w, *ws, *y;
    int64_t ldx, ldy, T, K, r, c;
    int32_t T32, K32, N, n_vis, block;
    float s_vis, s_txt;
    mquant_stream_t s;
    if (n != 9 || !read_rows(a[0], &x, &ldx, &T, &K) || !read_rows(a[8], &y, &ldy, &r, &c) || !read_size(T, &T32) ||
        !read_size(K, &K32) || !read_ptr(a[1], &w) || !read_ptr(a[2], &ws) || !read_i32(a[3], &N) ||
        !read_i32(a[4], &n_vis) || !read_f32(a[5], &s_vis) || !read_f32(a[6], &s_txt) || !read_i32(a[7], &block) ||
        !read_stream(m, &s))
        SLOW_WAY;
    LAUNCH(m->decode(x, ldx, w, ws, y, ldy, T32, N, K32, n_vis, s_vis, s_txt, block, s));
}

static PyObject *gemv_grouped(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    const State *m = PyModule_GetState(self);
    // xq, linears, n_vis, s_vis, s_txt
    void *xq;
    int64_t T, K;
    int32_t T32, K32, n_vis, count;
    float s_vis, s_txt;
    mquant_linear_t lin[4];
    mquant_stream_t s;
    if (n != 5 || a[0] == Py_None || !read_pair(PyObject_GetAttr(a[0], s_shape), &T, &K) || !read_dense(a[0], &xq) ||
        !read_size(T, &T32) || !read_size(K, &K32) || !read_linears(a[1], lin, &count) || !read_i32(a[2], &n_vis) ||
        !read_f32(a[3], &s_vis) || !read_f32(a[4], &s_txt) || !read_stream(m, &s))
        SLOW_WAY;
    LAUNCH(m->gemv_grouped(xq, T32, K32, n_vis, s_vis, s_txt, lin, count, s));
}

static PyObject *quant(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    const State *m = PyModule_GetState(self);
    // x, n_vis, s_vis, s_txt, had_block, perm, out
    void *x, *perm, *xq;
    int64_t ldx, T, K;
    int32_t T32, K32, n_vis, block;
    float s_vis, s_txt;
    mquant_stream_t s;
    if (n != 7 || !read_rows(a[0], &x, &ldx, &T, &K) || !read_size(T, &T32) || !read_size(K, &K32) ||
        !read_i32(a[1], &n_vis) || !read_f32(a[2], &s_vis) || !read_f32(a[3], &s_txt) || !read_i32(a[4], &block) ||
        !read_dense(a[5], &perm) || !read_dense(a[6], &xq) || !read_stream(m, &s))
        SLOW_WAY;
    LAUNCH(m->quant(x, ldx, perm, xq, T32, K32, n_vis, s_vis, s_txt, block, s));
}

static PyObject *weight_only(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    const State *m = PyModule_GetState(self);
    // x, w_prepacked, N, out; an empty x goes the slow way
    void *x, *w, *y;
    int64_t ldx, ldy, T, K, r, c;
    int32_t T32, K32, N;
    mquant_stream_t s;
    if (n != 4 || !read_rows(a[0], &x, &ldx, &T, &K) || !read_rows(a[3], &y, &ldy, &r, &c) || T == 0 ||
        !read_size(T, &T32) || !read_size(K, &K32) || !read_ptr(a[1], &w) || !read_i32(a[2], &N) || !read_stream(m, &s))
        SLOW_WAY;
    LAUNCH(m->weight_only(x, ldx, w, y, ldy, T32, N, K32, s));
}

// setup(is_initialized, device, raw stream, addresses of the seven entries of the library in the order of State)
static PyObject *setup(PyObject *self, PyObject *args)
{
    PyObject *init, *dev, *st, *addr[7];
    if (!PyArg_ParseTuple(args, "OOOO!O!O!O!O!O!O!", &init, &dev, &st, &PyLong_Type, &addr[0], &PyLong_Type, &addr[1],
                          &PyLong_Type, &addr[2], &PyLong_Type, &addr[3], &PyLong_Type, &addr[4], &PyLong_Type, &addr[5],
                          &PyLong_Type, &addr[6]))
        return NULL;
    void *p[7];
    for (int i = 0; i < 7; ++i) {
        p[i] = PyLong_AsVoidPtr(addr[i]);
        if (PyErr_Occurred()) return NULL;
    }
    State *m = PyModule_GetState(self);
    *(void **)&m->prefill = p[0];
    *(void **)&m->prefill_static = p[1];
    *(void **)&m->decode = p[2];
    *(void **)&m->decode_grouped = p[3];
    *(void **)&m->gemv_grouped = p[4];
    *(void **)&m->quant = p[5];
    *(void **)&m->weight_only = p[6];
    Py_INCREF(init), Py_INCREF(dev), Py_INCREF(st);
    Py_XSETREF(m->f_initialized, init);
    Py_XSETREF(m->f_device, dev);
    Py_XSETREF(m->f_stream, st);
    Py_RETURN_NONE;
}

#define ENTRY(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, NULL}
static PyMethodDef methods[] = {
    ENTRY(prefill), ENTRY(prefill_static), ENTRY(decode), ENTRY(decode_grouped), ENTRY(gemv_grouped), ENTRY(quant),
    ENTRY(weight_only), {"setup", setup, METH_VARARGS, NULL}, {NULL, NULL, 0, NULL},
};

static int traverse(PyObject *self, visitproc visit, void *arg)
{
    State *m = PyModule_GetState(self);
    Py_VISIT(m->f_initialized);
    Py_VISIT(m->f_device);
    Py_VISIT(m->f_stream);
    return 0;
}

static int clear(PyObject *self)
{
    State *m = PyModule_GetState(self);
    Py_CLEAR(m->f_stream);                     // first: a module without it takes no call
    Py_CLEAR(m->f_initialized);
    Py_CLEAR(m->f_device);
    return 0;
}

static int start(PyObject *self)
{
    s_shape = PyUnicode_InternFromString("shape");
    s_stride = PyUnicode_InternFromString("stride");
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_is_contiguous = PyUnicode_InternFromString("is_contiguous");
    return s_shape && s_stride && s_data_ptr && s_is_contiguous ? 0 : -1;
}

static PyModuleDef_Slot slots[] = {{Py_mod_exec, start}, {0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "mquant_fastcall", NULL, sizeof(State), methods, slots, traverse,
                                    clear, NULL};

PyMODINIT_FUNC PyInit_mquant_fastcall(void) { return PyModuleDef_Init(&module); }
