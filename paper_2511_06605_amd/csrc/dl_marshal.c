/*
 * Python argument marshalling of the calls that a program makes once per request: lists of tensors or addresses to
 * pointer arrays, tuples to copy descriptors, streams to handles.  Nothing else: the work is behind the dl_* entry
 * points, whose addresses binding.py hands over once (bind), so that whichever build of the library it has loaded is
 * the one that is called.  Done with ctypes objects this was most of a small request's time: all-gather of
 * 2 KiB over eight ranks 9.5 -> 7.2 us a call, 64 copies 21.6 -> 7.9, 256 copies 66.5 -> 10.5; with integers
 * of a list read where they lie, and the library taking them as plain copies, 64 / 256 / 900 copies 7.2 / 9.9 / 18.8 -> 6.7 / 7.6 /
 * 9.9.
 *
 * Arguments as the functions of binding.py take them: an address is an int, None (null) or an object with data_ptr();
 * a stream an int, None or an object with cuda_stream.  Every sequence (but a list or tuple of integer triples) is taken as a tuple first, so nothing that
 * runs in between (data_ptr() of a foreign class) can change what is being read, and the tuple is kept until the library
 * has returned: it may hold the only reference to a buffer (an iterator that makes tensors as it goes).  The lock of the
 * interpreter is released for the call into the library.
 */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>
#include <string.h>

#include "../../include/dmalatte.h"

enum { ON_STACK = 64 };

static struct {
    int (*allgather)(const void *const *, void *const *, int, size_t, void *);
    int (*alltoall)(const void *const *, void *const *, int, const size_t *, void *);
    int (*alltoall_inplace)(void *const *, int, size_t, void *);
    int (*broadcast)(const void *, void *const *, int, size_t, void *);
    int (*batch_copy)(const dl_copy_desc *, size_t, void *);
    int (*batch_copy_static)(const dl_copy_desc *, size_t, void *);
    int (*batch_swap)(const dl_swap_desc *, size_t, void *);
    int (*token_dispatch)(const void *const *, void *const *, int, const uint32_t *, size_t, const uint8_t *, void *);
    int (*token_dispatch_device)(const void *const *, void *const *, int, const uint32_t *, size_t, const uint8_t *, void *);
    int (*set_mode)(int);
    uint64_t (*last_ticket)(void);
    int (*trigger)(uint64_t);
    int (*wait)(uint64_t, uint64_t);
} lib;
static const char *const LIB_NAMES[] = {
    "dl_allgather", "dl_alltoall", "dl_alltoall_inplace", "dl_broadcast", "dl_batch_copy", "dl_batch_copy_static",
    "dl_batch_swap", "dl_token_dispatch", "dl_token_dispatch_device", "dl_set_mode", "dl_last_ticket", "dl_trigger", "dl_wait"};
enum { LIB_COUNT = sizeof LIB_NAMES / sizeof *LIB_NAMES };
_Static_assert(sizeof lib == LIB_COUNT * sizeof(void *), "one address per name");
_Static_assert(sizeof(dl_copy_desc) == 24 && sizeof(dl_swap_desc) == 24, "three words each");

static PyObject *s_data_ptr, *s_cuda_stream;

/* The value of an exact int of at most two digits of 30 bits (every address and length there is), read where it lies, for the
 * Pythons whose ints are known to lie that way.  0: x is something else. */
#if PY_VERSION_HEX < 0x030A0000
#include <longintrepr.h> /* later Python.h includes it, from 3.11 on under another name */
#endif
#if PY_VERSION_HEX < 0x030C0000 && PyLong_SHIFT == 30
enum { PLAIN_INTS = 1 };
static inline int plain_int(PyObject *x, uint64_t *out)
{
    if (!PyLong_CheckExact(x)) return 0;
    const Py_ssize_t digits = Py_SIZE(x);
    const digit *d = ((PyLongObject *)x)->ob_digit;
    if (digits == 2)
        *out = d[0] | (uint64_t)d[1] << PyLong_SHIFT;
    else if (digits == 1)
        *out = d[0];
    else if (digits == 0)
        *out = 0;
    else
        return 0;
    return 1;
}
#else
enum { PLAIN_INTS = 0 };
static inline int plain_int(PyObject *x, uint64_t *out) { return 0; }
#endif

/* int(x), reduced to 64 bits as ctypes does it */
static int to_u64(PyObject *x, uint64_t *out)
{
    if (plain_int(x, out)) return 0;
    if (PyLong_CheckExact(x)) {
        *out = PyLong_AsUnsignedLongLongMask(x);
        return *out == (uint64_t)-1 && PyErr_Occurred() ? -1 : 0;
    }
    PyObject *n = PyNumber_Long(x);
    if (!n) return -1;
    *out = PyLong_AsUnsignedLongLongMask(n);
    Py_DECREF(n);
    return *out == (uint64_t)-1 && PyErr_Occurred() ? -1 : 0;
}

static int to_address(PyObject *x, uint64_t *out)
{
    if (PyLong_CheckExact(x)) return to_u64(x, out);
    if (x == Py_None) {
        *out = 0;
        return 0;
    }
    PyObject *p = PyObject_CallMethodNoArgs(x, s_data_ptr);
    if (!p) {
        if (!PyErr_ExceptionMatches(PyExc_AttributeError)) return -1;
        /* no such method, or one that failed with this error itself? */
        PyObject *type, *value, *trace;
        PyErr_Fetch(&type, &value, &trace);
        if (PyObject_HasAttr(x, s_data_ptr)) {
            PyErr_Restore(type, value, trace);
            return -1;
        }
        Py_XDECREF(type);
        Py_XDECREF(value);
        Py_XDECREF(trace);
        return to_u64(x, out);
    }
    const int rc = to_u64(p, out);
    Py_DECREF(p);
    return rc;
}

static int to_stream(PyObject *x, void **out)
{
    uint64_t v = 0;
    int rc = 0;
    if (x != Py_None) {
        PyObject *h = PyLong_CheckExact(x) ? NULL : PyObject_GetAttr(x, s_cuda_stream);
        if (!h && PyErr_Occurred()) {
            if (!PyErr_ExceptionMatches(PyExc_AttributeError)) return -1;
            PyErr_Clear();
        }
        rc = to_u64(h ? h : x, &v);
        Py_XDECREF(h);
    }
    *out = (void *)(uintptr_t)v;
    return rc;
}

/* A sequence's values in an array: the caller's `room` of ON_STACK entries, or allocated; and what they are the
 * values of, for as long as the addresses are in use (free_values gives both up). */
typedef struct {
    uint64_t *v;
    Py_ssize_t n;
    PyObject *owners;
    uint64_t room[ON_STACK];
} values;

static void free_values(values *a)
{
    if (a->v != a->room) PyMem_Free(a->v);
    a->v = a->room;
    a->n = 0;
    Py_CLEAR(a->owners);
}

/* `a` is empty (free_values) before; to be given up by the caller in any case */
static int to_values(PyObject *seq, values *a, int (*convert)(PyObject *, uint64_t *))
{
    if (!(a->owners = PySequence_Tuple(seq))) return -1;
    const Py_ssize_t n = PyTuple_GET_SIZE(a->owners);
    if (n > ON_STACK && !(a->v = PyMem_New(uint64_t, n))) {
        a->v = a->room;
        PyErr_NoMemory();
        return -1;
    }
    for (; a->n < n; ++a->n)
        if (convert(PyTuple_GET_ITEM(a->owners, a->n), a->v + a->n) < 0) return -1;
    return 0;
}

static int want(Py_ssize_t have, Py_ssize_t n, const char *what)
{
    if (have == n) return lib.allgather ? 0 : (PyErr_SetString(PyExc_RuntimeError, "the library is not loaded"), -1);
    PyErr_Format(PyExc_TypeError, "%s takes %zd arguments", what, n);
    return -1;
}

#define UNLOCKED(rc, call)   \
    Py_BEGIN_ALLOW_THREADS   \
    (rc) = (call);           \
    Py_END_ALLOW_THREADS

static PyObject *m_allgather(PyObject *self, PyObject *const *args, Py_ssize_t n)
{
    values in = {.v = in.room}, out = {.v = out.room};
    uint64_t bytes;
    void *stream;
    PyObject *res = NULL;
    int rc;
    if (want(n, 4, "allgather") < 0) return NULL;
    if (to_values(args[0], &in, to_address) < 0 || to_values(args[1], &out, to_address) < 0) goto done;
    if (in.n != out.n) {
        PyErr_SetString(PyExc_ValueError, "need as many receive buffers as send buffers");
        goto done;
    }
    if (to_u64(args[2], &bytes) < 0 || to_stream(args[3], &stream) < 0) goto done;
    UNLOCKED(rc, lib.allgather((const void *const *)in.v, (void *const *)out.v, (int)in.n, (size_t)bytes, stream))
    res = PyLong_FromLong(rc);
done:
    free_values(&in);
    free_values(&out);
    return res;
}

static PyObject *m_alltoall(PyObject *self, PyObject *const *args, Py_ssize_t n)
{
    values in = {.v = in.room}, out = {.v = out.room}, row = {.v = row.room};
    uint64_t *chunks = NULL;
    Py_ssize_t have = 0, need;
    void *stream;
    PyObject *res = NULL, *rows = NULL;
    int rc;
    if (want(n, 4, "alltoall") < 0) return NULL;
    if (to_values(args[0], &in, to_address) < 0 || to_values(args[1], &out, to_address) < 0) goto done;
    if (in.n != out.n) {
        PyErr_SetString(PyExc_ValueError, "need as many receive buffers as send buffers");
        goto done;
    }
    need = in.n * in.n;
    if (!(rows = PySequence_Tuple(args[2])) || !(chunks = PyMem_New(uint64_t, need ? need : 1))) {
        if (rows) PyErr_NoMemory();
        goto done;
    }
    /* rows of W entries each, or the entries themselves */
    for (Py_ssize_t i = 0; i < PyTuple_GET_SIZE(rows); ++i) {
        PyObject *r = PyTuple_GET_ITEM(rows, i);
        free_values(&row);
        if (!PyLong_CheckExact(r) && PyObject_HasAttrString(r, "__len__")) {
            if (to_values(r, &row, to_u64) < 0) goto done;
        } else {
            if (to_u64(r, row.room) < 0) goto done;
            row.n = 1;
        }
        if (have + row.n <= need) memcpy(chunks + have, row.v, (size_t)row.n * sizeof *chunks);
        have += row.n;
    }
    if (have != need) {
        PyErr_SetString(PyExc_ValueError, "chunk_bytes must have W*W entries");
        goto done;
    }
    if (to_stream(args[3], &stream) < 0) goto done;
    UNLOCKED(rc, lib.alltoall((const void *const *)in.v, (void *const *)out.v, (int)in.n, (const size_t *)chunks, stream))
    res = PyLong_FromLong(rc);
done:
    Py_XDECREF(rows);
    PyMem_Free(chunks);
    free_values(&in);
    free_values(&out);
    free_values(&row);
    return res;
}

static PyObject *m_alltoall_inplace(PyObject *self, PyObject *const *args, Py_ssize_t n)
{
    values buf = {.v = buf.room};
    uint64_t bytes;
    void *stream;
    PyObject *res = NULL;
    int rc;
    if (want(n, 3, "alltoall_inplace") < 0) return NULL;
    if (to_values(args[0], &buf, to_address) == 0 && to_u64(args[1], &bytes) == 0 && to_stream(args[2], &stream) == 0) {
        UNLOCKED(rc, lib.alltoall_inplace((void *const *)buf.v, (int)buf.n, (size_t)bytes, stream))
        res = PyLong_FromLong(rc);
    }
    free_values(&buf);
    return res;
}

static PyObject *m_broadcast(PyObject *self, PyObject *const *args, Py_ssize_t n)
{
    values dst = {.v = dst.room};
    uint64_t src, bytes;
    void *stream;
    PyObject *res = NULL;
    int rc;
    if (want(n, 4, "broadcast") < 0) return NULL;
    if (to_address(args[0], &src) == 0 && to_values(args[1], &dst, to_address) == 0 && to_u64(args[2], &bytes) == 0 &&
        to_stream(args[3], &stream) == 0) {
        UNLOCKED(rc, lib.broadcast((const void *)(uintptr_t)src, (void *const *)dst.v, (int)dst.n, (size_t)bytes, stream))
        res = PyLong_FromLong(rc);
    }
    free_values(&dst);
    return res;
}

/* (address, address, bytes) triples, then the call */
static PyObject *triples(PyObject *const *args, Py_ssize_t n, const char *what, int which)
{
    PyObject *res = NULL, *t = NULL;
    uint64_t *w = NULL;
    Py_ssize_t count = 0;
    void *stream;
    int rc;
    if (want(n, 2, what) < 0) return NULL;
    /* a list or tuple of tuples of ints, as most are, is read where it lies (nothing else runs meanwhile, and ints keep no
     * buffer alive); with anything else in it, from its beginning as below */
    Py_ssize_t read = 0;
    if (PLAIN_INTS && (PyList_CheckExact(args[0]) || PyTuple_CheckExact(args[0]))) {
        const Py_ssize_t size = PySequence_Fast_GET_SIZE(args[0]);
        PyObject *const *const items = PySequence_Fast_ITEMS(args[0]);
        if (!(w = PyMem_New(uint64_t, 3 * (size ? size : 1)))) return PyErr_NoMemory();
        for (; read < size; ++read) {
            PyObject *d = items[read];
            if (!PyTuple_CheckExact(d) || PyTuple_GET_SIZE(d) != 3 || !plain_int(PyTuple_GET_ITEM(d, 0), w + 3 * read) ||
                !plain_int(PyTuple_GET_ITEM(d, 1), w + 3 * read + 1) || !plain_int(PyTuple_GET_ITEM(d, 2), w + 3 * read + 2))
                break;
        }
        if (read == size) {
            count = size;
            goto call;
        }
        PyMem_Free(w);
        w = NULL;
    }
    if (!(t = PySequence_Tuple(args[0]))) return NULL;
    count = PyTuple_GET_SIZE(t);
    if (!(w = PyMem_New(uint64_t, 3 * (count ? count : 1)))) {
        PyErr_NoMemory();
        goto done;
    }
    for (Py_ssize_t i = 0; i < count; ++i) {
        PyObject *d = PyTuple_GET_ITEM(t, i), *held = NULL;
        if (!PyTuple_CheckExact(d) && !(d = held = PySequence_Tuple(d))) goto done;
        int bad = PyTuple_GET_SIZE(d) != 3;
        if (bad)
            PyErr_Format(PyExc_ValueError, "%s: element %zd is not a triple", what, i);
        else
            bad = to_address(PyTuple_GET_ITEM(d, 0), w + 3 * i) < 0 || to_address(PyTuple_GET_ITEM(d, 1), w + 3 * i + 1) < 0 ||
                  to_u64(PyTuple_GET_ITEM(d, 2), w + 3 * i + 2) < 0;
        Py_XDECREF(held);
        if (bad) goto done;
    }
call:
    if (to_stream(args[1], &stream) < 0) goto done;
    Py_BEGIN_ALLOW_THREADS
    rc = which == 0   ? lib.batch_copy((const dl_copy_desc *)w, (size_t)count, stream)
         : which == 1 ? lib.batch_copy_static((const dl_copy_desc *)w, (size_t)count, stream)
                      : lib.batch_swap((const dl_swap_desc *)w, (size_t)count, stream);
    Py_END_ALLOW_THREADS
    res = PyLong_FromLong(rc);
done:
    PyMem_Free(w);
    Py_XDECREF(t);
    return res;
}

static PyObject *m_batch_copy(PyObject *self, PyObject *const *args, Py_ssize_t n) { return triples(args, n, "batch_copy", 0); }
static PyObject *m_batch_copy_static(PyObject *self, PyObject *const *args, Py_ssize_t n) { return triples(args, n, "batch_copy_static", 1); }
static PyObject *m_batch_swap(PyObject *self, PyObject *const *args, Py_ssize_t n) { return triples(args, n, "batch_swap", 2); }

/* The mask: a device address (on_device), or a C-contiguous buffer of one byte per (token, rank).  NotImplemented: the
 * host mask is not such a buffer; no other argument has been read, and the caller makes a buffer of it. */
static PyObject *dispatch(PyObject *const *args, Py_ssize_t n, const char *what, int on_device)
{
    values in = {.v = in.room}, out = {.v = out.room}, tok = {.v = tok.room};
    uint32_t on_stack[ON_STACK], *count = on_stack;
    uint64_t row, mask = 0, total = 0;
    Py_buffer view = {.obj = NULL};
    void *stream;
    PyObject *res = NULL;
    int rc;
    if (want(n, 6, what) < 0) return NULL;
    if (!on_device) {
        if (PyObject_GetBuffer(args[4], &view, PyBUF_C_CONTIGUOUS | PyBUF_FORMAT) < 0) {
            PyErr_Clear();
            return Py_NewRef(Py_NotImplemented);
        }
        if (view.itemsize != 1 || (view.format && !strchr("Bb?c", view.format[0]))) {
            res = Py_NewRef(Py_NotImplemented);
            goto done;
        }
        mask = (uint64_t)(uintptr_t)view.buf;
    }
    if (to_values(args[0], &in, to_address) < 0 || to_values(args[1], &out, to_address) < 0 || PyObject_Size(args[2]) < 0 ||
        to_values(args[2], &tok, to_u64) < 0)
        goto done;
    if (in.n != out.n || in.n != tok.n) {
        PyErr_SetString(PyExc_ValueError, "need W send buffers, W receive buffers and W token counts");
        goto done;
    }
    if (tok.n > ON_STACK && !(count = PyMem_New(uint32_t, tok.n))) {
        PyErr_NoMemory();
        goto done;
    }
    for (Py_ssize_t i = 0; i < tok.n; ++i) {
        total += tok.v[i];  /* the count as it was given: one that 32 bits do not hold goes with no mask */
        count[i] = (uint32_t)tok.v[i];
    }
    if (to_u64(args[3], &row) < 0) goto done;
    if (on_device) {
        if (to_address(args[4], &mask) < 0) goto done;
    } else if ((uint64_t)view.len != total * (uint64_t)in.n) {
        PyErr_SetString(PyExc_ValueError, "dest must have one entry per (token, rank)");
        goto done;
    }
    if (to_stream(args[5], &stream) < 0) goto done;
    Py_BEGIN_ALLOW_THREADS
    rc = (on_device ? lib.token_dispatch_device : lib.token_dispatch)((const void *const *)in.v, (void *const *)out.v, (int)in.n, count,
                                                                      (size_t)row, (const uint8_t *)(uintptr_t)mask, stream);
    Py_END_ALLOW_THREADS
    res = PyLong_FromLong(rc);
done:
    if (view.obj) PyBuffer_Release(&view);
    if (count != on_stack) PyMem_Free(count);
    free_values(&in);
    free_values(&out);
    free_values(&tok);
    return res;
}

static PyObject *m_token_dispatch(PyObject *self, PyObject *const *args, Py_ssize_t n) { return dispatch(args, n, "token_dispatch", 0); }
static PyObject *m_token_dispatch_device(PyObject *self, PyObject *const *args, Py_ssize_t n)
{
    return dispatch(args, n, "token_dispatch_device", 1);
}

/* Modes and tickets are whole numbers: an int or what stands for one (__index__).  Nothing else is converted here;
 * NotImplemented leaves it to the ctypes entry point, which refuses a text or a fraction and takes its own integers. */
static int to_whole(PyObject *x, uint64_t *out, PyObject **other)
{
    if (PyLong_CheckExact(x)) return to_u64(x, out);
    if (!PyIndex_Check(x)) {
        *other = Py_NewRef(Py_NotImplemented);
        return -1;
    }
    PyObject *n = PyNumber_Index(x);
    if (!n) return -1;
    const int rc = to_u64(n, out);
    Py_DECREF(n);
    return rc;
}

static PyObject *m_set_mode(PyObject *self, PyObject *const *args, Py_ssize_t n)
{
    PyObject *other = NULL;
    uint64_t mode;
    int rc;
    if (want(n, 1, "set_mode") < 0 || to_whole(args[0], &mode, &other) < 0) return other;
    UNLOCKED(rc, lib.set_mode((int)mode))
    return PyLong_FromLong(rc);
}

static PyObject *m_last_ticket(PyObject *self, PyObject *const *args, Py_ssize_t n)
{
    uint64_t t;
    if (want(n, 0, "last_ticket") < 0) return NULL;
    UNLOCKED(t, lib.last_ticket())
    return PyLong_FromUnsignedLongLong(t);
}

static PyObject *m_trigger(PyObject *self, PyObject *const *args, Py_ssize_t n)
{
    PyObject *other = NULL;
    uint64_t t;
    int rc;
    if (want(n, 1, "trigger") < 0 || to_whole(args[0], &t, &other) < 0) return other;
    UNLOCKED(rc, lib.trigger(t))
    return PyLong_FromLong(rc);
}

static PyObject *m_wait(PyObject *self, PyObject *const *args, Py_ssize_t n)
{
    PyObject *other = NULL;
    uint64_t t, ns;
    int rc;
    if (want(n, 2, "wait") < 0 || to_whole(args[0], &t, &other) < 0 || to_whole(args[1], &ns, &other) < 0) return other;
    UNLOCKED(rc, lib.wait(t, ns))
    return PyLong_FromLong(rc);
}

/* bind(addresses): of NAMES, in that order */
static PyObject *m_bind(PyObject *self, PyObject *seq)
{
    values a = {.v = a.room};
    PyObject *res = NULL;
    if (to_values(seq, &a, to_u64) == 0) {
        if (a.n != LIB_COUNT) {
            PyErr_SetString(PyExc_ValueError, "one address per name");
        } else {
            memcpy(&lib, a.v, sizeof lib);
            res = Py_NewRef(Py_None);
        }
    }
    free_values(&a);
    return res;
}

#define FAST(name) {#name, (PyCFunction)(void (*)(void))m_##name, METH_FASTCALL, NULL}
static PyMethodDef METHODS[] = {
    FAST(allgather), FAST(alltoall), FAST(alltoall_inplace), FAST(broadcast), FAST(batch_copy), FAST(batch_copy_static),
    FAST(batch_swap), FAST(token_dispatch), FAST(token_dispatch_device), FAST(set_mode), FAST(last_ticket), FAST(trigger),
    FAST(wait), {"bind", m_bind, METH_O, NULL}, {NULL, NULL, 0, NULL}};
static struct PyModuleDef MODULE = {PyModuleDef_HEAD_INIT, "_marshal", NULL, -1, METHODS, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__marshal(void)
{
    PyObject *m = PyModule_Create(&MODULE), *names = PyTuple_New(LIB_COUNT);
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    if (!m || !names || !s_data_ptr || !s_cuda_stream) return NULL;
    for (int i = 0; i < LIB_COUNT; ++i) {
        PyObject *s = PyUnicode_FromString(LIB_NAMES[i]);
        if (!s) return NULL;
        PyTuple_SET_ITEM(names, i, s);
    }
    return PyModule_AddObject(m, "NAMES", names) < 0 ? NULL : m;
}
