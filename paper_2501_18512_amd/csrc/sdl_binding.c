/* Argument marshalling of the device calls, as a Python extension module.
 *
 * The launch of a small call takes 4.5 us of the host, beside which the interpreter's share counts: every tensor asked for its device, its
 * layout and its address, the addresses packed, twelve arguments converted by ctypes.  Fused step of 2^16 parameters, 2 / 8 replicas
 * 6.2 / 8.3 us with that in Python and 4.8 / 6.2 here; the three calls of an exchange, 18.1 / 24.0 and 14.4 / 18.5.  Each function takes
 * the arguments of the binding's function of the same name, in that order, and returns the library's status.
 *
 * The rules are the binding's: a tensor has to be on a device and contiguous; None is a null pointer and an integer an address; what
 * is neither and has no is_cuda is asked for data_ptr() alone; a number is what ctypes takes for the argument's C type.  Nothing is kept from
 * one call for the next. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <stdint.h>
#include <string.h>

#include "sdl.h"

#define ENTRIES(X)                                                                                                          \
    X(sdl_quantize_outer_grad) X(sdl_dequant_reduce_nesterov) X(sdl_merge_overlap) X(sdl_receive_outer_step)                \
    X(sdl_fragment_outer_step) X(sdl_quantize_outer_grad_plan) X(sdl_dequant_reduce_nesterov_plan) X(sdl_merge_overlap_plan) \
    X(sdl_receive_outer_step_plan) X(sdl_fragment_outer_step_plan) X(sdl_fragment_outer_step_plan_static)                   \
    X(sdl_fragment_outer_step_plan_ex) X(sdl_fragment_outer_step_staged_ex)

/* the library's functions, by address (the library is loaded by the binding) */
#define DECLARE(name) static __typeof__(&name) p_##name;
ENTRIES(DECLARE)

static PyObject *s_is_cuda, *s_is_contiguous, *s_data_ptr, *s_h, *s_value;
static PyObject *f_stream, *f_initialized, *f_device, *f_raw_stream;
/* What ctypes makes of a value of a C type that is no plain integer or float: its own types, objects with _as_parameter_, ... or its
 * refusal.  f_packed: the same of an address in an array. */
static PyObject *t_void_p, *f_uint64, *f_uint32, *f_int, *f_float, *f_void_p, *f_packed;

static int address_by(PyObject* convert, PyObject* v, void** out)
{
    PyObject* r = v ? PyObject_CallOneArg(convert, v) : NULL;
    if (!r) return -1;
    *out = r == Py_None ? NULL : (void*)(uintptr_t)PyLong_AsUnsignedLongLongMask(r);
    Py_DECREF(r);
    return PyErr_Occurred() ? -1 : 0;
}

/* An address given as a value: of a single array, or of one in a list. */
static int address_of(PyObject* v, int in_list, void** out)
{
    if (!PyLong_Check(v)) return address_by(in_list ? f_packed : f_void_p, v, out);
    *out = in_list ? PyLong_AsVoidPtr(v) : (void*)(uintptr_t)PyLong_AsUnsignedLongLongMask(v);
    if (!PyErr_Occurred()) return 0;
    PyErr_Clear();
    return address_by(f_packed, v, out);
}

/* The address of a tensor, checked. */
static int address(PyObject* t, int in_list, void** out)
{
    PyObject *v, *w;
    int on_device, contiguous;
    if (t == Py_None) {
        *out = NULL;
        return 0;
    }
    if (PyLong_Check(t)) return address_of(t, in_list, out);
    v = PyObject_GetAttr(t, s_is_cuda);
    w = v ? PyObject_CallMethodNoArgs(t, s_is_contiguous) : NULL;
    if (w) {
        on_device = PyObject_IsTrue(v);
        contiguous = PyObject_IsTrue(w);
        Py_DECREF(v);
        Py_DECREF(w);
        if (on_device < 0 || contiguous < 0) return -1;
        if (!on_device || !contiguous) {
            PyErr_SetString(PyExc_ValueError, on_device ? "sdl calls take contiguous tensors"
                                                        : "sdl calls take device tensors; there is no CPU path");
            return -1;
        }
    } else {
        Py_XDECREF(v);
        if (!PyErr_ExceptionMatches(PyExc_AttributeError)) return -1;
        PyErr_Clear();
    }
    v = PyObject_CallMethodNoArgs(t, s_data_ptr);
    if (!v) return -1;
    on_device = address_of(v, in_list, out);
    Py_DECREF(v);
    return on_device;
}

/* The addresses of several; null behind them.  More than the library takes are looked at, for the library to refuse their number.
 * What is walked is a tuple of them: looking at a tensor may run Python code, in which a caller's list may change. */
typedef struct {
    void* at[SDL_MAX_WORKERS];
    void** p;
    Py_ssize_t n;
} Addresses;

static int addresses(PyObject* ts, Addresses* a)
{
    PyObject* items;
    Py_ssize_t i;
    void* unused;
    a->p = NULL;
    a->n = 0;
    memset(a->at, 0, sizeof(a->at));
    if (ts == Py_None) return 0;
    items = PySequence_Tuple(ts);
    if (!items) return -1;
    a->n = PyTuple_GET_SIZE(items);
    for (i = 0; i < a->n; ++i)
        if (address(PyTuple_GET_ITEM(items, i), 1, i < SDL_MAX_WORKERS ? &a->at[i] : &unused) < 0) {
            Py_DECREF(items);
            return -1;
        }
    Py_DECREF(items);
    a->p = a->at;
    return 0;
}

/* How many they were; what has no length (None, a generator) is refused. */
static int count(PyObject* ts, const Addresses* a, uint32_t* out)
{
    if (PyObject_Length(ts) < 0) return -1;
    *out = (uint32_t)a->n;
    return 0;
}

static int whole(PyObject* v, PyObject* convert, uint64_t* out)
{
    PyObject* r = PyLong_Check(v) ? NULL : PyObject_CallOneArg(convert, v);
    if (!r && PyErr_Occurred()) return -1;
    *out = PyLong_AsUnsignedLongLongMask(r ? r : v);
    Py_XDECREF(r);
    return PyErr_Occurred() ? -1 : 0;
}

static int real(PyObject* v, float* out)
{
    PyObject* r = NULL;
    double d = PyFloat_Check(v) || PyLong_Check(v) ? PyFloat_AsDouble(v) : -1.0;
    if (!PyFloat_Check(v) && (!PyLong_Check(v) || PyErr_Occurred())) {
        PyErr_Clear();
        r = PyObject_CallOneArg(f_float, v);
        if (!r) return -1;
        d = PyFloat_AsDouble(r);
        Py_DECREF(r);
    }
    *out = (float)d;
    return PyErr_Occurred() ? -1 : 0;
}

/* The handle that an owner (a Plan) holds; NULL once it has been given back. */
static int handle(PyObject* owner, void** out)
{
    int rc;
    PyObject* h = PyObject_GetAttr(owner, s_h);
    if (h && (PyObject*)Py_TYPE(h) == t_void_p) {
        PyObject* v = PyObject_GetAttr(h, s_value);
        Py_DECREF(h);
        h = v;
    }
    if (!h) return -1;
    *out = NULL;
    rc = h == Py_None ? 0 : address_of(h, 0, out);
    Py_DECREF(h);
    return rc;
}

/* The stream's handle: what the binding's _stream returns, for the current stream without going through the interpreter. */
static int stream_of(PyObject* s, void** out)
{
    PyObject *v = NULL, *d;
    int rc = 0;
    if (s == Py_None && f_raw_stream != Py_None) {
        v = PyObject_CallNoArgs(f_initialized);
        if (!v) return -1;
        if (v == Py_True) {
            Py_DECREF(v);
            d = PyObject_CallNoArgs(f_device);
            if (!d) return -1;
            v = PyObject_CallOneArg(f_raw_stream, d);
            Py_DECREF(d);
            if (!v) return -1;
        } else {
            Py_DECREF(v);
            v = NULL;
        }
    }
    if (!v && !(v = PyObject_CallOneArg(f_stream, s))) return -1;
    *out = NULL;
    if (v != Py_None) rc = address_of(v, 0, out);
    Py_DECREF(v);
    return rc;
}

static int argc_is(Py_ssize_t n, Py_ssize_t want)
{
    if (n == want) return 1;
    PyErr_Format(PyExc_TypeError, "%zd arguments, not %zd", want, n);
    return 0;
}

/* The library is called without the interpreter's lock. */
#define CALL(expression)                  \
    do {                                  \
        int status;                       \
        Py_BEGIN_ALLOW_THREADS            \
        status = (expression);            \
        Py_END_ALLOW_THREADS              \
        return PyLong_FromLong(status);   \
    } while (0)

#define FUNCTION(name) static PyObject* b_##name(PyObject* self, PyObject* const* a, Py_ssize_t n)
#define W(x) ((const void* const*)(x).p)
#define V(x) ((void* const*)(x).p)

FUNCTION(sdl_quantize_outer_grad)        /* g, w_send, n, fmt, codes, scales, stream */
{
    void *g, *st;
    Addresses w, c, s;
    uint32_t M;
    uint64_t numel, fmt;
    if (!argc_is(n, 7) || address(a[0], 0, &g) || addresses(a[1], &w) || addresses(a[4], &c) || addresses(a[5], &s) || count(a[1], &w, &M)
        || whole(a[2], f_uint64, &numel) || whole(a[3], f_int, &fmt) || stream_of(a[6], &st)) return NULL;
    CALL(p_sdl_quantize_outer_grad(g, W(w), M, numel, (sdl_format_t)fmt, V(c), V(s), st));
}

FUNCTION(sdl_dequant_reduce_nesterov)    /* g, mom, codes, scales, n, fmt, lr, mu, stream */
{
    void *g, *mom, *st;
    Addresses c, s;
    uint32_t M;
    uint64_t numel, fmt;
    float lr, mu;
    if (!argc_is(n, 9) || address(a[0], 0, &g) || address(a[1], 0, &mom) || addresses(a[2], &c) || addresses(a[3], &s) || count(a[2], &c, &M)
        || whole(a[4], f_uint64, &numel) || whole(a[5], f_int, &fmt) || real(a[6], &lr) || real(a[7], &mu) || stream_of(a[8], &st)) return NULL;
    CALL(p_sdl_dequant_reduce_nesterov(g, mom, W(c), W(s), M, numel, (sdl_format_t)fmt, lr, mu, st));
}

FUNCTION(sdl_merge_overlap)              /* g_new, w_now, n, alpha, stream */
{
    void *g, *st;
    Addresses w;
    uint32_t M;
    uint64_t numel;
    float alpha;
    if (!argc_is(n, 5) || address(a[0], 0, &g) || addresses(a[1], &w) || count(a[1], &w, &M) || whole(a[2], f_uint64, &numel) || real(a[3], &alpha)
        || stream_of(a[4], &st)) return NULL;
    CALL(p_sdl_merge_overlap(g, V(w), M, numel, alpha, st));
}

FUNCTION(sdl_receive_outer_step)         /* g, mom, codes, scales, w_now, n, fmt, lr, mu, alpha, stream */
{
    void *g, *mom, *st;
    Addresses c, s, w;
    uint32_t M, M_c;
    uint64_t numel, fmt;
    float lr, mu, alpha;
    if (!argc_is(n, 11) || address(a[0], 0, &g) || address(a[1], 0, &mom) || addresses(a[2], &c) || addresses(a[3], &s) || addresses(a[4], &w)
        || count(a[2], &c, &M_c) || count(a[4], &w, &M)) return NULL;
    if (M != M_c) return PyLong_FromLong(SDL_ERR_INVALID_ARG);
    if (whole(a[5], f_uint64, &numel) || whole(a[6], f_int, &fmt) || real(a[7], &lr) || real(a[8], &mu) || real(a[9], &alpha) || stream_of(a[10], &st)) return NULL;
    CALL(p_sdl_receive_outer_step(g, mom, W(c), W(s), V(w), M, numel, (sdl_format_t)fmt, lr, mu, alpha, st));
}

FUNCTION(sdl_fragment_outer_step)        /* g, mom, w_send, w_now, n, fmt, lr, mu, alpha, codes, scales, stream */
{
    void *g, *mom, *st;
    Addresses ws, wn, c, s;
    uint32_t M, M_now;
    uint64_t numel, fmt;
    float lr, mu, alpha;
    if (!argc_is(n, 12) || address(a[0], 0, &g) || address(a[1], 0, &mom) || addresses(a[2], &ws) || addresses(a[3], &wn) || addresses(a[9], &c)
        || addresses(a[10], &s) || count(a[2], &ws, &M) || count(a[3], &wn, &M_now)) return NULL;
    if (M != M_now) return PyLong_FromLong(SDL_ERR_INVALID_ARG);
    if (whole(a[4], f_uint64, &numel) || whole(a[5], f_int, &fmt) || real(a[6], &lr) || real(a[7], &mu) || real(a[8], &alpha) || stream_of(a[11], &st)) return NULL;
    CALL(p_sdl_fragment_outer_step(g, mom, W(ws), V(wn), M, numel, (sdl_format_t)fmt, lr, mu, alpha, V(c), V(s), st));
}

FUNCTION(sdl_quantize_outer_grad_plan)   /* plan, p, g, w_send, fmt, codes, scales, stream */
{
    void *plan, *g, *st;
    Addresses w, c, s;
    uint32_t M;
    uint64_t p, fmt;
    if (!argc_is(n, 8) || address(a[2], 0, &g) || addresses(a[3], &w) || addresses(a[5], &c) || addresses(a[6], &s) || handle(a[0], &plan)
        || whole(a[1], f_uint32, &p) || count(a[3], &w, &M) || whole(a[4], f_int, &fmt) || stream_of(a[7], &st)) return NULL;
    CALL(p_sdl_quantize_outer_grad_plan(plan, (uint32_t)p, g, W(w), M, (sdl_format_t)fmt, V(c), V(s), st));
}

FUNCTION(sdl_dequant_reduce_nesterov_plan)   /* plan, p, g, mom, codes, scales, fmt, lr, mu, stream */
{
    void *plan, *g, *mom, *st;
    Addresses c, s;
    uint32_t M;
    uint64_t p, fmt;
    float lr, mu;
    if (!argc_is(n, 10) || address(a[2], 0, &g) || address(a[3], 0, &mom) || addresses(a[4], &c) || addresses(a[5], &s) || handle(a[0], &plan)
        || whole(a[1], f_uint32, &p) || count(a[4], &c, &M) || whole(a[6], f_int, &fmt) || real(a[7], &lr) || real(a[8], &mu) || stream_of(a[9], &st)) return NULL;
    CALL(p_sdl_dequant_reduce_nesterov_plan(plan, (uint32_t)p, g, mom, W(c), W(s), M, (sdl_format_t)fmt, lr, mu, st));
}

FUNCTION(sdl_merge_overlap_plan)         /* plan, p, g_new, w_now, alpha, stream */
{
    void *plan, *g, *st;
    Addresses w;
    uint32_t M;
    uint64_t p;
    float alpha;
    if (!argc_is(n, 6) || address(a[2], 0, &g) || addresses(a[3], &w) || handle(a[0], &plan) || whole(a[1], f_uint32, &p) || count(a[3], &w, &M)
        || real(a[4], &alpha) || stream_of(a[5], &st)) return NULL;
    CALL(p_sdl_merge_overlap_plan(plan, (uint32_t)p, g, V(w), M, alpha, st));
}

FUNCTION(sdl_receive_outer_step_plan)    /* plan, p, g, mom, codes, scales, w_now, fmt, lr, mu, alpha, stream */
{
    void *plan, *g, *mom, *st;
    Addresses c, s, w;
    uint32_t M;
    uint64_t p, fmt;
    float lr, mu, alpha;
    if (!argc_is(n, 12) || address(a[2], 0, &g) || address(a[3], 0, &mom) || addresses(a[4], &c) || addresses(a[5], &s) || addresses(a[6], &w)
        || handle(a[0], &plan) || whole(a[1], f_uint32, &p) || count(a[6], &w, &M) || whole(a[7], f_int, &fmt) || real(a[8], &lr) || real(a[9], &mu) || real(a[10], &alpha)
        || stream_of(a[11], &st)) return NULL;
    CALL(p_sdl_receive_outer_step_plan(plan, (uint32_t)p, g, mom, W(c), W(s), V(w), M, (sdl_format_t)fmt, lr, mu, alpha, st));
}

/* plan, p, g, mom, w_send, w_now, fmt, lr, mu, alpha and, at the end, stream */
typedef struct {
    void *plan, *g, *mom, *st;
    Addresses ws, wn;
    uint32_t M, p;
    sdl_format_t fmt;
    float lr, mu, alpha;
} Step;

/* -1: an exception is set; 1: the two lists differ in length (which the staged form has never looked at: what w_now lacks is null, which
 * the library refuses, and what it has beyond w_send is not read) */
static int step_args(PyObject* const* a, PyObject* stream, int staged, PyObject* codes, PyObject* scales, Addresses* c, Addresses* s, Step* x)
{
    uint32_t M_now;
    uint64_t p, fmt;
    if (address(a[2], 0, &x->g) || address(a[3], 0, &x->mom) || addresses(a[4], &x->ws) || addresses(a[5], &x->wn)
        || (codes && (addresses(codes, c) || addresses(scales, s))) || count(a[4], &x->ws, &x->M) || (!staged && count(a[5], &x->wn, &M_now))) return -1;
    if (!staged && x->M != M_now) return 1;
    if (handle(a[0], &x->plan) || whole(a[1], f_uint32, &p) || whole(a[6], f_int, &fmt) || real(a[7], &x->lr) || real(a[8], &x->mu) || real(a[9], &x->alpha)
        || stream_of(stream, &x->st)) return -1;
    x->p = (uint32_t)p;
    x->fmt = (sdl_format_t)fmt;
    return 0;
}

FUNCTION(sdl_fragment_outer_step_plan)
{
    Step x;
    int rc = argc_is(n, 11) ? step_args(a, a[10], 0, NULL, NULL, NULL, NULL, &x) : -1;
    if (rc) return rc < 0 ? NULL : PyLong_FromLong(SDL_ERR_INVALID_ARG);
    CALL(p_sdl_fragment_outer_step_plan(x.plan, x.p, x.g, x.mom, W(x.ws), V(x.wn), x.M, x.fmt, x.lr, x.mu, x.alpha, x.st));
}

FUNCTION(sdl_fragment_outer_step_plan_static)
{
    Step x;
    int rc = argc_is(n, 11) ? step_args(a, a[10], 0, NULL, NULL, NULL, NULL, &x) : -1;
    if (rc) return rc < 0 ? NULL : PyLong_FromLong(SDL_ERR_INVALID_ARG);
    CALL(p_sdl_fragment_outer_step_plan_static(x.plan, x.p, x.g, x.mom, W(x.ws), V(x.wn), x.M, x.fmt, x.lr, x.mu, x.alpha, x.st));
}

FUNCTION(sdl_fragment_outer_step_plan_ex)    /* ..., codes, scales, stream */
{
    Step x;
    Addresses c, s;
    int rc = argc_is(n, 13) ? step_args(a, a[12], 0, a[10], a[11], &c, &s, &x) : -1;
    if (rc) return rc < 0 ? NULL : PyLong_FromLong(SDL_ERR_INVALID_ARG);
    CALL(p_sdl_fragment_outer_step_plan_ex(x.plan, x.p, x.g, x.mom, W(x.ws), V(x.wn), x.M, x.fmt, x.lr, x.mu, x.alpha, V(c), V(s), x.st));
}

FUNCTION(sdl_fragment_outer_step_staged_ex)  /* ..., codes, scales, stream */
{
    Step x;
    Addresses c, s;
    int rc = argc_is(n, 13) ? step_args(a, a[12], 1, a[10], a[11], &c, &s, &x) : -1;
    if (rc) return rc < 0 ? NULL : PyLong_FromLong(SDL_ERR_INVALID_ARG);
    CALL(p_sdl_fragment_outer_step_staged_ex(x.plan, x.p, x.g, x.mom, W(x.ws), V(x.wn), x.M, x.fmt, x.lr, x.mu, x.alpha, V(c), V(s), x.st));
}

/* The library's functions by name (a dict of addresses), then the binding's _stream, and what it asks for the current stream. */
static PyObject* setup(PyObject* self, PyObject* args)
{
    PyObject *by_name, *at;
    if (!PyArg_ParseTuple(args, "O!OOOO", &PyDict_Type, &by_name, &f_stream, &f_initialized, &f_device, &f_raw_stream)) return NULL;
    Py_INCREF(f_stream);
    Py_INCREF(f_initialized);
    Py_INCREF(f_device);
    Py_INCREF(f_raw_stream);
#define TAKE(name)                                                             \
    at = PyDict_GetItemString(by_name, #name);                                 \
    if (!at) return PyErr_Format(PyExc_KeyError, "%s", #name);                 \
    p_##name = (__typeof__(&name))PyLong_AsVoidPtr(at);                        \
    if (!p_##name) return PyErr_Occurred() ? NULL : PyErr_Format(PyExc_ValueError, "%s", #name);
    ENTRIES(TAKE)
    Py_RETURN_NONE;
}

/* ctypes.c_void_p, then the conversions in the order of their declaration */
static PyObject* converters(PyObject* self, PyObject* args)
{
    PyObject** const all[] = {&t_void_p, &f_uint64, &f_uint32, &f_int, &f_float, &f_void_p, &f_packed};
    size_t i;
    if (!PyArg_ParseTuple(args, "OOOOOOO", all[0], all[1], all[2], all[3], all[4], all[5], all[6])) return NULL;
    for (i = 0; i < sizeof(all) / sizeof(all[0]); ++i) Py_INCREF(*all[i]);
    Py_RETURN_NONE;
}

#define METHOD(name) {#name, (PyCFunction)(void (*)(void))b_##name, METH_FASTCALL, NULL},
static PyMethodDef methods[] = {{"setup", setup, METH_VARARGS, NULL}, {"converters", converters, METH_VARARGS, NULL}, ENTRIES(METHOD) {NULL, NULL, 0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__binding(void)
{
    s_is_cuda = PyUnicode_InternFromString("is_cuda");
    s_is_contiguous = PyUnicode_InternFromString("is_contiguous");
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_h = PyUnicode_InternFromString("_h");
    s_value = PyUnicode_InternFromString("value");
    if (!s_is_cuda || !s_is_contiguous || !s_data_ptr || !s_h || !s_value) return NULL;
    return PyModule_Create(&module);
}
