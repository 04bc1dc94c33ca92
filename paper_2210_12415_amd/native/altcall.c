/* The calls a program repeats, marshalled natively: descriptors and layouts by the address of their ctypes object, tensors by data_ptr(), the
 * current stream by its number.  A function returns the library's status, or None where an argument is not of the plain types below; the
 * caller then takes the call through ctypes, which decides as ever what it accepts and what it raises.  (An interrupt, or whatever else is no
 * Exception, that ends an argument's own code is raised at once: the second attempt would not see it again.) */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stddef.h>
#include <stdint.h>
#include <unistd.h>

enum { CONV2D, CONV3D, CONV2D_TRANSPOSE, CONV3D_TRANSPOSE, GEMM, TRANSFORM, ADD, FUNCTIONS };

typedef int (*operator_fn)(void *, const void *, const void *, const void *, const float *, void *, void *, size_t, void *);
typedef int (*gemm_fn)(void *, const void *, const void *, const void *, void *, void *, size_t, void *);
typedef int (*transform_fn)(void *, int, int, const int64_t *, const void *, const void *, const void *, void *, void *);
typedef int (*add_fn)(void *, int, int64_t, const void *, const void *, void *, int, void *);

static void *entry[FUNCTIONS];
static PyObject *handle_type, *conv_type, *conv3d_type, *gemm_type, *layout_type;
static PyObject *raw_stream, *get_device;                  /* torch's, once it has initialised the device */
static pid_t stream_pid;
static PyObject *s_data_ptr, *s_cuda_stream;

/* An argument is not taken: its exception goes, for ctypes to raise.  -1 */
static int refused(void)
{
    if (PyErr_Occurred() && PyErr_ExceptionMatches(PyExc_Exception)) PyErr_Clear();
    return -1;
}

/* The answer for arguments that are not taken. */
static PyObject *not_taken(void)
{
    if (PyErr_Occurred()) return NULL;
    Py_RETURN_NONE;
}

/* 0, or -1 for an object of another type. */
static int object_at(PyObject *o, PyObject *type, void **out)
{
    Py_buffer b;
    if ((PyObject *)Py_TYPE(o) != type) return -1;
    if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) return refused();
    *out = b.buf;
    PyBuffer_Release(&b);
    return 0;
}

static int number(PyObject *o, unsigned long long most, unsigned long long *out)
{
    if (!PyLong_CheckExact(o)) return -1;
    *out = PyLong_AsUnsignedLongLong(o);
    if (*out == (unsigned long long)-1 && PyErr_Occurred()) return refused();
    return *out <= most ? 0 : -1;
}

static int number_of(PyObject *r, void **out)              /* takes the reference; NULL: an exception is set */
{
    unsigned long long v;
    if (!r) return refused();
    const int bad = number(r, UINT64_MAX, &v);
    Py_DECREF(r);
    *out = (void *)(uintptr_t)v;
    return bad;
}

static int address(PyObject *o, void **out)
{
    unsigned long long v;
    if (o == Py_None) { *out = NULL; return 0; }
    if (PyLong_CheckExact(o)) {
        if (number(o, UINT64_MAX, &v) != 0) return -1;
        *out = (void *)(uintptr_t)v;
        return 0;
    }
    return number_of(PyObject_CallMethodNoArgs(o, s_data_ptr), out);
}

static int stream_of(PyObject *o, void **out)
{
    if (o == Py_None) {
        if (!raw_stream || getpid() != stream_pid) return -1;
        PyObject *d = PyObject_CallNoArgs(get_device);
        if (!d) return refused();
        PyObject *r = PyObject_CallOneArg(raw_stream, d);
        Py_DECREF(d);
        return number_of(r, out);
    }
    if (PyLong_CheckExact(o)) return address(o, out);
    return number_of(PyObject_GetAttr(o, s_cuda_stream), out);
}

static int handle_of(PyObject *o, void **out)
{
    void *at;
    if (object_at(o, handle_type, &at) != 0) return -1;
    *out = *(void **)at;
    return 0;
}

typedef struct {
    void *h, *d, *x, *w, *bias, *y, *workspace, *stream;
    size_t ws_bytes;
} operator_args;

/* (h, d, x, w, bias, y, workspace, ws_bytes, stream); all but h */
static int operator_args_of(PyObject *const *a, PyObject *type, operator_args *r)
{
    unsigned long long ws;
    if (object_at(a[1], type, &r->d) || address(a[2], &r->x) || address(a[3], &r->w) || address(a[4], &r->bias) ||
        address(a[5], &r->y) || address(a[6], &r->workspace) || number(a[7], SIZE_MAX, &ws) || stream_of(a[8], &r->stream))
        return -1;
    r->ws_bytes = (size_t)ws;
    return 0;
}

static int call_operator(int which, const operator_args *r)
{
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = ((operator_fn)entry[which])(r->h, r->d, r->x, r->w, (const float *)r->bias, r->y, r->workspace, r->ws_bytes, r->stream);
    Py_END_ALLOW_THREADS
    return status;
}

static PyObject *operator_call(int which, PyObject *type, PyObject *const *a, Py_ssize_t n)
{
    operator_args r;
    if (n != 9 || !entry[which] || handle_of(a[0], &r.h) || operator_args_of(a, type, &r)) return not_taken();
    return PyLong_FromLong(call_operator(which, &r));
}

static PyObject *py_conv2d(PyObject *m, PyObject *const *a, Py_ssize_t n) { return operator_call(CONV2D, conv_type, a, n); }
static PyObject *py_conv3d(PyObject *m, PyObject *const *a, Py_ssize_t n) { return operator_call(CONV3D, conv3d_type, a, n); }
static PyObject *py_conv2d_transpose(PyObject *m, PyObject *const *a, Py_ssize_t n) { return operator_call(CONV2D_TRANSPOSE, conv_type, a, n); }
static PyObject *py_conv3d_transpose(PyObject *m, PyObject *const *a, Py_ssize_t n) { return operator_call(CONV3D_TRANSPOSE, conv3d_type, a, n); }

/* (h, d, A, B, C, workspace, ws_bytes, stream) */
static PyObject *py_gemm(PyObject *m, PyObject *const *a, Py_ssize_t n)
{
    void *h, *d, *A, *B, *C, *ws, *st;
    unsigned long long bytes;
    int status;
    if (n != 8 || !entry[GEMM] || handle_of(a[0], &h) || object_at(a[1], gemm_type, &d) || address(a[2], &A) || address(a[3], &B) ||
        address(a[4], &C) || address(a[5], &ws) || number(a[6], SIZE_MAX, &bytes) || stream_of(a[7], &st))
        return not_taken();
    Py_BEGIN_ALLOW_THREADS
    status = ((gemm_fn)entry[GEMM])(h, d, A, B, C, ws, (size_t)bytes, st);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

/* (h, dtype, shape, src_layout, src, dst_layout, dst, stream) */
static PyObject *py_layout_transform(PyObject *m, PyObject *const *a, Py_ssize_t n)
{
    void *h, *ls, *ld, *src, *dst, *st;
    unsigned long long dtype, v;
    int64_t shape[16];
    int status;
    if (n != 8 || !entry[TRANSFORM] || handle_of(a[0], &h) || number(a[1], 255, &dtype) || !PyTuple_CheckExact(a[2])) return not_taken();
    const Py_ssize_t nd = PyTuple_GET_SIZE(a[2]);
    if (nd > 16) return not_taken();
    for (Py_ssize_t i = 0; i < nd; ++i) {
        if (number(PyTuple_GET_ITEM(a[2], i), INT64_MAX, &v)) return not_taken();
        shape[i] = (int64_t)v;
    }
    if (object_at(a[3], layout_type, &ls) || address(a[4], &src) || object_at(a[5], layout_type, &ld) || address(a[6], &dst) || stream_of(a[7], &st))
        return not_taken();
    Py_BEGIN_ALLOW_THREADS
    status = ((transform_fn)entry[TRANSFORM])(h, (int)dtype, (int)nd, shape, ls, src, ld, dst, st);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

/* (h, dtype, numel, a, b, y, relu, stream) */
static PyObject *py_eltwise_add(PyObject *m, PyObject *const *a, Py_ssize_t n)
{
    void *h, *x, *y, *z, *st;
    unsigned long long dtype, numel;
    int status;
    if (n != 8 || !entry[ADD] || handle_of(a[0], &h) || number(a[1], 255, &dtype) || number(a[2], INT64_MAX, &numel) || address(a[3], &x) ||
        address(a[4], &y) || address(a[5], &z) || !PyBool_Check(a[6]) || stream_of(a[7], &st))
        return not_taken();
    const int relu = a[6] == Py_True;
    Py_BEGIN_ALLOW_THREADS
    status = ((add_fn)entry[ADD])(h, (int)dtype, (int64_t)numel, x, y, z, relu, st);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

/* A call of conv2d with its arguments marshalled once.  It keeps what they came from, the owner of the handle among them. */
typedef struct {
    PyObject_HEAD
    vectorcallfunc vectorcall;
    PyObject *handle, *keep, *failed;                      /* failed(status, handle) raises */
    operator_args r;
} Prepared;

static PyObject *prepared_call(PyObject *self, PyObject *const *a, size_t n, PyObject *kw)
{
    Prepared *p = (Prepared *)self;
    if (PyVectorcall_NARGS(n) != 0 || (kw && PyTuple_GET_SIZE(kw) != 0)) {
        PyErr_SetString(PyExc_TypeError, "a prepared call takes no arguments");
        return NULL;
    }
    operator_args r = p->r;
    if (handle_of(p->handle, &r.h)) r.h = NULL;
    const int status = call_operator(CONV2D, &r);
    if (status != 0) {
        PyObject *s = PyObject_CallFunction(p->failed, "iO", status, p->handle);
        if (!s) return NULL;
        Py_DECREF(s);
    }
    Py_RETURN_FALSE;
}

static int prepared_traverse(PyObject *self, visitproc visit, void *arg)
{
    Prepared *p = (Prepared *)self;
    Py_VISIT(p->handle); Py_VISIT(p->keep); Py_VISIT(p->failed);
    return 0;
}

static int prepared_clear(PyObject *self)
{
    Prepared *p = (Prepared *)self;
    Py_CLEAR(p->handle); Py_CLEAR(p->keep); Py_CLEAR(p->failed);
    return 0;
}

static void prepared_dealloc(PyObject *self)
{
    PyObject_GC_UnTrack(self);
    prepared_clear(self);
    PyObject_GC_Del(self);
}

static PyTypeObject prepared_type = {
    PyVarObject_HEAD_INIT(NULL, 0).tp_name = "paper_2210_12415_amd.PreparedCall", .tp_basicsize = sizeof(Prepared),
    .tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_GC | Py_TPFLAGS_HAVE_VECTORCALL, .tp_vectorcall_offset = offsetof(Prepared, vectorcall),
    .tp_call = PyVectorcall_Call, .tp_traverse = prepared_traverse, .tp_clear = prepared_clear, .tp_dealloc = prepared_dealloc,
};

/* (h, d, x, w, bias, y, workspace, ws_bytes, stream, failed, the owner of h) */
static PyObject *py_prepare_conv2d(PyObject *m, PyObject *const *a, Py_ssize_t n)
{
    operator_args r;
    if (n != 11 || !entry[CONV2D] || handle_of(a[0], &r.h) || operator_args_of(a, conv_type, &r)) return not_taken();
    PyObject *keep = PyTuple_Pack(7, a[10], a[1], a[2], a[3], a[4], a[5], a[6]);
    if (!keep) return NULL;
    Prepared *p = PyObject_GC_New(Prepared, &prepared_type);
    if (!p) { Py_DECREF(keep); return NULL; }
    p->vectorcall = prepared_call;
    p->handle = a[0]; Py_INCREF(a[0]);
    p->failed = a[9]; Py_INCREF(a[9]);
    p->keep = keep;
    p->r = r;
    PyObject_GC_Track((PyObject *)p);
    return (PyObject *)p;
}

/* (the seven entry points' addresses, then the types of handles, of the three descriptors and of layouts) */
static PyObject *py_setup(PyObject *m, PyObject *const *a, Py_ssize_t n)
{
    if (n != FUNCTIONS + 5) { PyErr_SetString(PyExc_TypeError, "setup: wrong number of arguments"); return NULL; }
    void *at[FUNCTIONS];
    for (int i = 0; i < FUNCTIONS; ++i) {
        at[i] = PyLong_AsVoidPtr(a[i]);
        if (PyErr_Occurred()) return NULL;
    }
    PyObject **types[5] = {&handle_type, &conv_type, &conv3d_type, &gemm_type, &layout_type};
    for (int i = 0; i < 5; ++i) { Py_INCREF(a[FUNCTIONS + i]); Py_XSETREF(*types[i], a[FUNCTIONS + i]); }
    for (int i = 0; i < FUNCTIONS; ++i) entry[i] = at[i];
    Py_RETURN_NONE;
}

/* (the current stream's number of a device, the current device): in the process that initialised the GPU */
static PyObject *py_streams(PyObject *m, PyObject *const *a, Py_ssize_t n)
{
    if (n != 2) { PyErr_SetString(PyExc_TypeError, "streams: wrong number of arguments"); return NULL; }
    Py_INCREF(a[0]); Py_XSETREF(raw_stream, a[0]);
    Py_INCREF(a[1]); Py_XSETREF(get_device, a[1]);
    stream_pid = getpid();
    Py_RETURN_NONE;
}

#define FAST(name) {#name, (PyCFunction)(void (*)(void))py_##name, METH_FASTCALL, NULL}
static PyMethodDef methods[] = {FAST(conv2d), FAST(conv3d), FAST(conv2d_transpose), FAST(conv3d_transpose), FAST(gemm), FAST(layout_transform),
                                FAST(eltwise_add), FAST(prepare_conv2d), FAST(setup), FAST(streams), {NULL, NULL, 0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_altcall", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__altcall(void)
{
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    if (!s_data_ptr || !s_cuda_stream || PyType_Ready(&prepared_type) < 0) return NULL;
    return PyModule_Create(&module);
}
