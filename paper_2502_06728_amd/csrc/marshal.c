/* Argument marshalling of the Python binding for the calls a program makes on every step.
 *
 * A step on a small shard is shorter on the GPU than the type and length checks, attribute reads
 * and ctypes conversions of its two calls are in Python (1 Mi parameters: some 10 us of kernels
 * behind 21 us of Python).  These functions do the same reads and checks in C.  They take a call
 * on only if everything is as usual (contiguous device tensors of the right types and lengths,
 * a valid configuration, no debug output, no explicit strides) and return -1 otherwise: the
 * caller then goes through the binding's own checks, which say what is wrong.  No tensor data is
 * touched here; the status of the library call is returned as it is.
 */
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <stdint.h>

#include "../../include/detonation.h"

typedef int (*compress_fn)(const deto_config*, int64_t, const void*, int, float*, void*, int, void*,
                           int, float*, void*);
typedef int (*decompress_fn)(const deto_config*, int64_t, int32_t, const void*, int, int64_t,
                             const void*, int, int64_t, void*, int, float*, void*);
typedef int (*adamw_fn)(const deto_config*, const deto_adamw*, int64_t, int32_t, const void*, int,
                        int64_t, const void*, int, int64_t, void*, int, float*, float*, float*,
                        float*, void*);

static compress_fn call_compress;
static decompress_fn call_decompress;
static adamw_fn call_adamw;

/* torch's dtype objects, in the order of enum dt (borrowed forever: they are never freed) */
enum dt { DT_F32, DT_BF16, DT_F16, DT_I32, DT_U8, DT_COUNT };
static PyObject* dtypes[DT_COUNT];

/* torch's functions for the current device and the raw handle of its current stream */
static PyObject *fn_device, *fn_stream;

static PyObject *s_chunk, *s_topk, *s_scheme, *s_sign, *s_dct, *s_decay, *s_lr, *s_weight_decay,
    *s_seed, *s_step, *s_beta1, *s_beta2, *s_eps, *s_amsgrad, *s_is_cuda, *s_is_contiguous, *s_numel,
    *s_dtype, *s_data_ptr;

static int get_long(PyObject* o, PyObject* name, long long* out) {
    PyObject* v = PyObject_GetAttr(o, name);
    if (!v) return 0;
    *out = PyLong_Check(v) ? PyLong_AsLongLong(v) : -1;
    const int ok = PyLong_Check(v) && !PyErr_Occurred();
    Py_DECREF(v);
    return ok;
}

static int get_u64(PyObject* o, PyObject* name, uint64_t* out) {   /* wraps, as ctypes does */
    PyObject* v = PyObject_GetAttr(o, name);
    if (!v) return 0;
    const int ok = PyLong_Check(v);
    if (ok) *out = PyLong_AsUnsignedLongLongMask(v);
    Py_DECREF(v);
    return ok && !PyErr_Occurred();
}

static int get_float(PyObject* o, PyObject* name, float* out) {
    PyObject* v = PyObject_GetAttr(o, name);
    if (!v) return 0;
    *out = (float)PyFloat_AsDouble(v);
    Py_DECREF(v);
    return !PyErr_Occurred();
}

static int get_truth(PyObject* o, PyObject* name, int* out) {
    PyObject* v = PyObject_GetAttr(o, name);
    if (!v) return 0;
    *out = PyObject_IsTrue(v);
    Py_DECREF(v);
    return *out >= 0;
}

static int get_config(PyObject* o, deto_config* c) {
    long long chunk, topk, scheme;
    int sign, dct;
    if (!get_long(o, s_chunk, &chunk) || !get_long(o, s_topk, &topk) ||
        !get_long(o, s_scheme, &scheme) || !get_truth(o, s_sign, &sign) ||
        !get_truth(o, s_dct, &dct) || !get_float(o, s_decay, &c->decay) ||
        !get_float(o, s_lr, &c->lr) || !get_float(o, s_weight_decay, &c->weight_decay) ||
        !get_u64(o, s_seed, &c->seed) || !get_u64(o, s_step, &c->step))
        return 0;
    if (topk < 1 || topk > chunk || chunk > 256 || scheme < 0 || scheme > 2) return 0;
    c->chunk = (int32_t)chunk;
    c->topk = (int32_t)topk;
    c->scheme = (int32_t)scheme;
    c->flags = (sign ? DETO_FLAG_SIGN : 0u) | (dct ? DETO_FLAG_DCT : 0u);
    return 1;
}

static int call_long(PyObject* o, PyObject* method, long long* out) {
    PyObject* v = PyObject_CallMethodNoArgs(o, method);
    if (!v) return 0;
    *out = PyLong_AsLongLong(v);
    Py_DECREF(v);
    return !PyErr_Occurred();
}

/* a contiguous device tensor: its type, length and address */
static int get_tensor(PyObject* t, int* dt, long long* numel, void** ptr) {
    int cuda, contiguous;
    if (!get_truth(t, s_is_cuda, &cuda) || !cuda) return 0;
    PyObject* v = PyObject_CallMethodNoArgs(t, s_is_contiguous);
    if (!v) return 0;
    contiguous = PyObject_IsTrue(v);
    Py_DECREF(v);
    if (contiguous <= 0) return 0;
    v = PyObject_GetAttr(t, s_dtype);
    if (!v) return 0;
    for (*dt = 0; *dt < DT_COUNT; ++*dt)
        if (dtypes[*dt] == v) break;
    Py_DECREF(v);
    if (*dt == DT_COUNT) return 0;
    v = PyObject_CallMethodNoArgs(t, s_data_ptr);
    if (!v) return 0;
    *ptr = PyLong_AsVoidPtr(v);
    Py_DECREF(v);
    return !PyErr_Occurred() && call_long(t, s_numel, numel);
}

/* idx / val of `replicas` contiguous payloads */
struct payload {
    void *idx, *val;
    int idx_dtype, val_dtype;
    int64_t entries, val_elems;
};

static int get_payload(const deto_config* c, int64_t n, PyObject* idx, PyObject* val,
                       long long replicas, int packed, struct payload* p) {
    const int64_t chunks = (n + c->chunk - 1) / c->chunk;
    long long numel;
    int dt;
    p->entries = chunks * c->topk;
    if (!get_tensor(val, &dt, &numel, &p->val) || dt == DT_U8 || (!packed && dt != DT_F32)) return 0;
    p->val_dtype = dt == DT_F32 ? DETO_F32 : dt == DT_BF16 ? DETO_BF16 : dt == DT_F16 ? DETO_F16
                                                                                     : DETO_TERNARY;
    p->val_elems = dt == DT_I32 ? chunks * ((c->topk + 15) / 16) : p->entries;
    if (numel / replicas < p->val_elems) return 0;
    p->idx = NULL;
    p->idx_dtype = DETO_IDX_I32;
    if (idx == Py_None) return c->scheme != DETO_SCHEME_TOPK;
    if (!get_tensor(idx, &dt, &numel, &p->idx) || !(dt == DT_I32 || (packed && dt == DT_U8))) return 0;
    p->idx_dtype = dt == DT_U8 ? DETO_IDX_U8 : DETO_IDX_I32;
    return numel / replicas >= p->entries;
}

static int get_n(PyObject* given, PyObject* like, long long* n) {
    if (given == Py_None) return call_long(like, s_numel, n);
    if (!PyLong_Check(given)) return 0;
    *n = PyLong_AsLongLong(given);
    return !PyErr_Occurred();
}

/* a stream handle, or None: the current stream of the current device */
static int get_stream(PyObject* given, void** out) {
    if (given == Py_None) {
        PyObject* dev = PyObject_CallNoArgs(fn_device);
        if (!dev) return 0;
        PyObject* h = PyObject_CallOneArg(fn_stream, dev);
        Py_DECREF(dev);
        if (!h) return 0;
        *out = PyLong_AsVoidPtr(h);
        Py_DECREF(h);
    } else {
        *out = PyLong_AsVoidPtr(given);
    }
    return !PyErr_Occurred();
}

static PyObject* unusual(void) {
    PyErr_Clear();
    return PyLong_FromLong(-1);
}

/* compress(cfg, n, grad, momentum, idx_out, val_out, packed, stream) */
static PyObject* py_compress(PyObject* self, PyObject* const* a, Py_ssize_t count) {
    (void)self;
    deto_config c;
    struct payload p;
    long long n, g_len, m_len;
    int g_dt, m_dt, rc;
    void *g, *m, *stream;
    if (count != 8 || !get_n(a[1], a[3], &n) || n < 0 || !get_config(a[0], &c) ||
        !get_tensor(a[2], &g_dt, &g_len, &g) || (g_dt != DT_F32 && g_dt != DT_BF16) || g_len < n ||
        !get_tensor(a[3], &m_dt, &m_len, &m) || m_dt != DT_F32 || m_len < n ||
        !get_payload(&c, n, a[4], a[5], 1, a[6] == Py_True, &p) || !get_stream(a[7], &stream))
        return unusual();
    Py_BEGIN_ALLOW_THREADS
    rc = call_compress(&c, n, g, g_dt == DT_BF16 ? DETO_BF16 : DETO_F32, (float*)m, p.idx,
                       p.idx_dtype, p.val, p.val_dtype, NULL, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

/* decompress(cfg, n, R, idx, val, params, packed, stream[, opt, exp_avg, exp_avg_sq, max]) */
static PyObject* py_decompress(PyObject* self, PyObject* const* a, Py_ssize_t count) {
    (void)self;
    deto_config c;
    deto_adamw o;
    struct payload p;
    long long n, len, R;
    int dt, t_dt, rc;
    void *theta, *stream, *moment[3] = {NULL, NULL, NULL};
    if ((count != 8 && count != 12) || !PyLong_Check(a[2])) return unusual();
    R = PyLong_AsLongLong(a[2]);
    if (PyErr_Occurred() || R < 1 || R > INT32_MAX || !get_n(a[1], a[5], &n) || n < 0 ||
        !get_config(a[0], &c) || !get_tensor(a[5], &t_dt, &len, &theta) ||
        (t_dt != DT_F32 && t_dt != DT_BF16) || len < n ||
        !get_payload(&c, n, a[3], a[4], R, a[6] == Py_True, &p))
        return unusual();
    if (count == 12) {
        long long amsgrad;
        if (!get_float(a[8], s_beta1, &o.beta1) || !get_float(a[8], s_beta2, &o.beta2) ||
            !get_float(a[8], s_eps, &o.eps) || !get_long(a[8], s_amsgrad, &amsgrad) ||
            (amsgrad != 0 && amsgrad != 1) || !get_u64(a[8], s_step, &o.step))
            return unusual();
        o.amsgrad = (int32_t)amsgrad;
        for (int i = 0; i < 3; ++i) {
            if (i == 2 && a[11] == Py_None && !amsgrad) continue;
            if (!get_tensor(a[9 + i], &dt, &len, &moment[i]) || dt != DT_F32 || len < n)
                return unusual();
        }
    }
    if (!get_stream(a[7], &stream)) return unusual();
    const int p_dt = t_dt == DT_BF16 ? DETO_BF16 : DETO_F32;
    Py_BEGIN_ALLOW_THREADS
    if (count == 12)
        rc = call_adamw(&c, &o, n, (int32_t)R, p.idx, p.idx_dtype, p.entries, p.val, p.val_dtype,
                        p.val_elems, theta, p_dt, (float*)moment[0], (float*)moment[1],
                        (float*)moment[2], NULL, stream);
    else
        rc = call_decompress(&c, n, (int32_t)R, p.idx, p.idx_dtype, p.entries, p.val, p.val_dtype,
                             p.val_elems, theta, p_dt, NULL, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

/* setup(addresses of the three packed entry points, torch dtypes in the order of enum dt, current
 * device, current stream of a device) */
static PyObject* py_setup(PyObject* self, PyObject* args) {
    (void)self;
    unsigned long long f[3];
    PyObject *d[DT_COUNT], *device, *stream;
    if (!PyArg_ParseTuple(args, "KKKOOOOOOO", &f[0], &f[1], &f[2], &d[0], &d[1], &d[2], &d[3], &d[4],
                          &device, &stream))
        return NULL;
    Py_INCREF(device);
    Py_INCREF(stream);
    Py_XSETREF(fn_device, device);
    Py_XSETREF(fn_stream, stream);
    call_compress = (compress_fn)(uintptr_t)f[0];
    call_decompress = (decompress_fn)(uintptr_t)f[1];
    call_adamw = (adamw_fn)(uintptr_t)f[2];
    for (int i = 0; i < DT_COUNT; ++i) {
        Py_INCREF(d[i]);
        Py_XSETREF(dtypes[i], d[i]);
    }
    Py_RETURN_NONE;
}

static PyMethodDef methods[] = {
    {"setup", py_setup, METH_VARARGS, "entry points and torch's dtypes"},
    {"compress", (PyCFunction)(void (*)(void))py_compress, METH_FASTCALL, "status, or -1"},
    {"decompress", (PyCFunction)(void (*)(void))py_decompress, METH_FASTCALL, "status, or -1"},
    {NULL, NULL, 0, NULL}};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", NULL, -1, methods,
                                    NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__marshal(void) {
    struct { PyObject** at; const char* name; } names[] = {
        {&s_chunk, "chunk"}, {&s_topk, "topk"}, {&s_scheme, "scheme"}, {&s_sign, "sign"},
        {&s_dct, "dct"}, {&s_decay, "decay"}, {&s_lr, "lr"}, {&s_weight_decay, "weight_decay"},
        {&s_seed, "seed"}, {&s_step, "step"}, {&s_beta1, "beta1"}, {&s_beta2, "beta2"},
        {&s_eps, "eps"}, {&s_amsgrad, "amsgrad"}, {&s_is_cuda, "is_cuda"},
        {&s_is_contiguous, "is_contiguous"}, {&s_numel, "numel"}, {&s_dtype, "dtype"},
        {&s_data_ptr, "data_ptr"}};
    for (size_t i = 0; i < sizeof(names) / sizeof(names[0]); ++i)
        if (!(*names[i].at = PyUnicode_InternFromString(names[i].name))) return NULL;
    return PyModule_Create(&module);
}
