// The binding's argument marshalling in native code: what a training step passes on every call -
// lists of tensors or pointer tables, the update rule's tuple, a plan, the current stream - turned
// into the C ABI's arguments without a ctypes object per argument.  A small round runs for 4 us on
// the GPU; through ctypes the calls of one step (plan, round) took 10 us of Python.
//
// Every function here returns NotImplemented for arguments of a form it does not know (anything
// but the exact types named below); the binding then takes the ctypes path, which defines what
// is accepted and how it is refused.  Nothing is computed here and nothing is kept between calls.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include "../../include/eager.h"

#include <limits.h>
#include <stdint.h>

namespace {

struct Entry {                       // the library's entry points, handed over by the binding
    decltype(&eager_plan_participation) plan_participation;
    decltype(&eager_plan_quorum) plan_quorum;
    decltype(&eager_partial_allreduce_solo) rounds[3];      // solo, majority, quorum
    decltype(&eager_partial_allreduce_lagging) lagging;
    decltype(&eager_partial_allreduce_exchange) exchange;
    decltype(&eager_sgd_step) sgd;
    decltype(&eager_sgd_step_lars) lars;
    decltype(&eager_stash) stash;
    decltype(&eager_sgd_step_views) views;
    decltype(&eager_average_views) average;
};
Entry lib;
PyObject *plan_type, *array_type, *get_device, *get_stream;
PyObject *s_data_ptr, *s_cuda_stream;

// true: the form is known and `out` is set.  false with no error set: another form.
bool as_pointer(PyObject *x, void **out)
{
    if (x == Py_None) {
        *out = nullptr;
        return true;
    }
    PyObject *v = x;
    if (PyLong_Check(x)) {
        Py_INCREF(v);
    } else {
        v = PyObject_CallMethodNoArgs(x, s_data_ptr);       // a torch tensor
        if (!v) return false;
        if (!PyLong_Check(v)) {
            Py_DECREF(v);
            return false;
        }
    }
    const unsigned long long p = PyLong_AsUnsignedLongLong(v);
    Py_DECREF(v);
    if (p == static_cast<unsigned long long>(-1) && PyErr_Occurred()) {
        PyErr_Clear();                                      // negative or too large
        return false;
    }
    *out = reinterpret_cast<void *>(p);
    return true;
}

bool as_int(PyObject *x, int *out)
{
    if (!PyLong_CheckExact(x)) return false;
    int over = 0;
    const long v = PyLong_AsLongAndOverflow(x, &over);
    if (over || v < INT_MIN || v > INT_MAX) return false;
    *out = static_cast<int>(v);
    return true;
}

bool as_u64(PyObject *x, uint64_t *out)
{
    if (!PyLong_CheckExact(x)) return false;
    *out = PyLong_AsUnsignedLongLongMask(x);                // modulo 2^64, as ctypes does
    return true;
}

bool as_float(PyObject *x, float *out)
{
    if (!PyFloat_CheckExact(x)) return false;
    *out = static_cast<float>(PyFloat_AS_DOUBLE(x));
    return true;
}

// b1: None means the last bucket
bool as_range(PyObject *b0, PyObject *b1, PyObject *n_buckets, int *lo, int *hi)
{
    return as_int(b0, lo) && as_int(b1 == Py_None ? n_buckets : b1, hi);
}

// None: torch's current stream of the current device, asked for as torch.cuda.current_stream does
bool as_stream(PyObject *x, void **out)
{
    if (x != Py_None) {
        if (PyLong_Check(x)) return as_pointer(x, out);
        PyObject *v = PyObject_GetAttr(x, s_cuda_stream);
        if (!v) return false;
        const bool ok = PyLong_Check(v) && as_pointer(v, out);
        Py_DECREF(v);
        return ok;
    }
    if (!get_stream) return false;                          // torch's GPU side not initialised yet
    PyObject *dev = PyObject_CallNoArgs(get_device);
    if (!dev) return false;
    PyObject *v = PyObject_CallOneArg(get_stream, dev);
    Py_DECREF(dev);
    if (!v) return false;
    const bool ok = PyLong_Check(v) && as_pointer(v, out);
    Py_DECREF(v);
    return ok;
}

// A pointer table: a ctypes array of c_void_p (used in place, so that the library can exchange
// entries in it), or a list or tuple whose pointers are collected here.
struct Table {
    void *own[EAGER_MAX_P];
    void **p = nullptr;
    int n = 0;
    Py_buffer view{};
    bool held = false;
    ~Table()
    {
        if (held) PyBuffer_Release(&view);
    }
    bool in_place() const { return held; }
    bool take(PyObject *x)
    {
        if (PyList_CheckExact(x) || PyTuple_CheckExact(x)) {
            const Py_ssize_t len = PySequence_Fast_GET_SIZE(x);
            if (len > EAGER_MAX_P) return false;
            for (Py_ssize_t i = 0; i < len; ++i) {
                if (i >= PySequence_Fast_GET_SIZE(x)) return false;
                PyObject *e = PySequence_Fast_GET_ITEM(x, i);
                Py_INCREF(e);
                const bool ok = as_pointer(e, &own[i]);
                Py_DECREF(e);
                if (!ok) return false;
            }
            p = own;
            n = static_cast<int>(len);
            return true;
        }
        if (PyObject_IsInstance(x, array_type) != 1) return false;
        if (PyObject_GetBuffer(x, &view, PyBUF_FORMAT | PyBUF_WRITABLE) != 0) {
            PyErr_Clear();
            return false;
        }
        held = true;
        if (view.itemsize != 8 || !view.format || view.len % 8 != 0 || view.len / 8 > EAGER_MAX_P) return false;
        const char *f = view.format;
        while (f[0] && f[1]) ++f;
        if (*f != 'P') return false;
        p = static_cast<void **>(view.buf);
        n = static_cast<int>(view.len / 8);
        return true;
    }
};

// (params, momentum, lr, mu)
bool as_opt(PyObject *x, eager_opt *opt)
{
    void *w = nullptr, *v = nullptr;
    if (!PyTuple_CheckExact(x) || PyTuple_GET_SIZE(x) != 4) return false;
    if (!as_pointer(PyTuple_GET_ITEM(x, 0), &w) || !as_pointer(PyTuple_GET_ITEM(x, 1), &v) ||
        !as_float(PyTuple_GET_ITEM(x, 2), &opt->lr) || !as_float(PyTuple_GET_ITEM(x, 3), &opt->mu))
        return false;
    opt->params = static_cast<float *>(w);
    opt->momentum = static_cast<float *>(v);
    return true;
}

PyObject *other_form()
{
    if (PyErr_Occurred()) return nullptr;                   // raised by a caller's object: as it is
    Py_RETURN_NOTIMPLEMENTED;
}

bool arrivals(PyObject *x, double (&t)[EAGER_MAX_P], int *P)
{
    if (!PyList_CheckExact(x) && !PyTuple_CheckExact(x)) return false;
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(x);
    if (n < 1 || n > EAGER_MAX_P) return false;
    for (Py_ssize_t i = 0; i < n; ++i) {
        PyObject *e = PySequence_Fast_GET_ITEM(x, i);
        if (!PyFloat_CheckExact(e)) return false;
        t[i] = PyFloat_AS_DOUBLE(e);
    }
    *P = static_cast<int>(n);
    return true;
}

// a new Plan, or the status
PyObject *plan_object(int status, const eager_plan &plan)
{
    if (status != EAGER_OK) return PyLong_FromLong(status);
    PyObject *o = PyObject_CallNoArgs(plan_type);
    if (!o) return nullptr;
    Py_buffer view;
    if (PyObject_GetBuffer(o, &view, PyBUF_WRITABLE) != 0) {
        Py_DECREF(o);
        return nullptr;
    }
    if (view.len == static_cast<Py_ssize_t>(sizeof plan)) *static_cast<eager_plan *>(view.buf) = plan;
    PyBuffer_Release(&view);
    return o;
}

// plan_participation(mode, arrival_ms, seed, step, window_ms, flags)
PyObject *py_plan_participation(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    int mode, P, flags;
    uint64_t seed, step;
    double t[EAGER_MAX_P];
    if (n != 6 || !as_int(a[0], &mode) || !arrivals(a[1], t, &P) || !as_u64(a[2], &seed) ||
        !as_u64(a[3], &step) || !PyFloat_CheckExact(a[4]) || !as_int(a[5], &flags))
        return other_form();
    eager_plan plan;
    const int st = lib.plan_participation(mode, P, t, seed, step, PyFloat_AS_DOUBLE(a[4]),
                                          static_cast<uint32_t>(flags), &plan);
    return plan_object(st, plan);
}

// plan_quorum(arrival_ms, quorum, step, window_ms)
PyObject *py_plan_quorum(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    int P, quorum;
    uint64_t step;
    double t[EAGER_MAX_P];
    if (n != 4 || !arrivals(a[0], t, &P) || !as_int(a[1], &quorum) || !as_u64(a[2], &step) ||
        !PyFloat_CheckExact(a[3]))
        return other_form();
    eager_plan plan;
    const int st = lib.plan_quorum(P, t, quorum, step, PyFloat_AS_DOUBLE(a[3]), &plan);
    return plan_object(st, plan);
}

// round(kind, ctx, P, n_buckets, plan, absent, b0, b1, grads, resid, recv, opt, stream)
// kind: 0..2 the modes, 3 lagging, 4 exchange
PyObject *py_round(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    int kind, P, b0, b1;
    uint64_t absent;
    void *ctx, *recv, *stream;
    eager_opt opt;
    if (n != 13 || !as_int(a[0], &kind) || kind < 0 || kind > 4 || !as_pointer(a[1], &ctx) || !as_int(a[2], &P) ||
        !Py_IS_TYPE(a[4], reinterpret_cast<PyTypeObject *>(plan_type)) || !as_u64(a[5], &absent) ||
        !as_range(a[6], a[7], a[3], &b0, &b1))
        return other_form();
    Table g, r;
    if (!g.take(a[8]) || !r.take(a[9]) || g.n != P || r.n != P || !as_pointer(a[10], &recv)) return other_form();
    if (kind == 4 && (!g.in_place() || !r.in_place())) return other_form();
    if (a[11] != Py_None && !as_opt(a[11], &opt)) return other_form();
    if (!as_stream(a[12], &stream)) return other_form();
    Py_buffer plan_view;
    if (PyObject_GetBuffer(a[4], &plan_view, PyBUF_SIMPLE) != 0) return nullptr;
    const eager_plan plan = *static_cast<const eager_plan *>(plan_view.buf);
    PyBuffer_Release(&plan_view);
    const eager_opt *o = a[11] == Py_None ? nullptr : &opt;
    eager_ctx *c = static_cast<eager_ctx *>(ctx);
    const void *const *grads = const_cast<const void *const *>(g.p);
    float *const *resid = reinterpret_cast<float *const *>(r.p);
    float *out = static_cast<float *>(recv);
    int st;
    Py_BEGIN_ALLOW_THREADS
    if (kind == 3)
        st = lib.lagging(c, &plan, absent, b0, b1, grads, resid, out, o, stream);
    else if (kind == 4)
        st = lib.exchange(c, &plan, const_cast<const void **>(g.p), reinterpret_cast<float **>(r.p), out, o, stream);
    else
        st = lib.rounds[kind](c, &plan, b0, b1, grads, resid, out, o, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
}

// step(ctx, n_buckets, b0, b1, update, opt, trust, eps, stream): trust None = the plain rule
PyObject *py_step(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    int b0, b1;
    void *ctx, *update, *stream;
    eager_opt opt;
    float trust = 0.0f, eps = 0.0f;
    if (n != 9 || !as_pointer(a[0], &ctx) || !as_range(a[2], a[3], a[1], &b0, &b1) || !as_pointer(a[4], &update) ||
        !as_opt(a[5], &opt) || (a[6] != Py_None && (!as_float(a[6], &trust) || !as_float(a[7], &eps))) ||
        !as_stream(a[8], &stream))
        return other_form();
    const bool layerwise = a[6] != Py_None;
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = layerwise ? lib.lars(static_cast<eager_ctx *>(ctx), b0, b1, static_cast<float *>(update), &opt, trust, eps, stream)
                   : lib.sgd(static_cast<eager_ctx *>(ctx), b0, b1, static_cast<float *>(update), &opt, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
}

// stash(ctx, n_buckets, process, b0, b1, grad, resid, stream)
PyObject *py_stash(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    int process, b0, b1;
    void *ctx, *grad, *resid, *stream;
    if (n != 8 || !as_pointer(a[0], &ctx) || !as_int(a[2], &process) || !as_range(a[3], a[4], a[1], &b0, &b1) ||
        !as_pointer(a[5], &grad) || !as_pointer(a[6], &resid) || !as_stream(a[7], &stream))
        return other_form();
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = lib.stash(static_cast<eager_ctx *>(ctx), process, b0, b1, grad, static_cast<float *>(resid), stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
}

// views(ctx, n_buckets, b0, b1, update, params, momentum, lr, mu, stream); momentum None = average
PyObject *py_views(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    int b0, b1;
    void *ctx, *update, *stream;
    float lr = 0.0f, mu = 0.0f;
    Table w, v;
    if (n != 10 || !as_pointer(a[0], &ctx) || !as_range(a[2], a[3], a[1], &b0, &b1) || !as_pointer(a[4], &update) ||
        !w.take(a[5]) || !as_stream(a[9], &stream))
        return other_form();
    const bool average = a[6] == Py_None;
    // (the number of views is the length of the parameter table; a shorter momentum table is not
    // for this path)
    if (!average && (!v.take(a[6]) || v.n != w.n || !as_float(a[7], &lr) || !as_float(a[8], &mu))) return other_form();
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = average ? lib.average(static_cast<eager_ctx *>(ctx), b0, b1, w.n, reinterpret_cast<float *const *>(w.p), stream)
                 : lib.views(static_cast<eager_ctx *>(ctx), b0, b1, static_cast<float *>(update), w.n,
                             reinterpret_cast<float *const *>(w.p), reinterpret_cast<float *const *>(v.p), lr, mu, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
}

// bind(addresses, Plan, ctypes.Array)
PyObject *py_bind(PyObject *, PyObject *args)
{
    PyObject *addr, *plan, *array;
    if (!PyArg_ParseTuple(args, "O!OO", &PyTuple_Type, &addr, &plan, &array)) return nullptr;
    constexpr Py_ssize_t kN = sizeof(Entry) / sizeof(void *);
    if (PyTuple_GET_SIZE(addr) != kN) {
        PyErr_SetString(PyExc_ValueError, "one address per entry point");
        return nullptr;
    }
    void *p[kN];
    for (Py_ssize_t i = 0; i < kN; ++i) {
        p[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(addr, i));
        if (!p[i]) return PyErr_Occurred() ? nullptr : PyErr_Format(PyExc_ValueError, "entry point %zd is NULL", i);
    }
    __builtin_memcpy(&lib, p, sizeof lib);
    Py_INCREF(plan);
    Py_INCREF(array);
    Py_XSETREF(plan_type, plan);
    Py_XSETREF(array_type, array);
    Py_RETURN_NONE;
}

// streams(get_device, get_stream): torch's functions, or None, None to forget them
PyObject *py_streams(PyObject *, PyObject *args)
{
    PyObject *dev, *str;
    if (!PyArg_ParseTuple(args, "OO", &dev, &str)) return nullptr;
    if (str == Py_None) {
        Py_CLEAR(get_device);
        Py_CLEAR(get_stream);
    } else {
        Py_INCREF(dev);
        Py_INCREF(str);
        Py_XSETREF(get_device, dev);
        Py_XSETREF(get_stream, str);
    }
    Py_RETURN_NONE;
}

#define FAST(f) reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL
PyMethodDef methods[] = {
    {"bind", py_bind, METH_VARARGS, nullptr},
    {"streams", py_streams, METH_VARARGS, nullptr},
    {"plan_participation", FAST(py_plan_participation), nullptr},
    {"plan_quorum", FAST(py_plan_quorum), nullptr},
    {"round", FAST(py_round), nullptr},
    {"step", FAST(py_step), nullptr},
    {"stash", FAST(py_stash), nullptr},
    {"views", FAST(py_views), nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void)
{
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    if (!s_data_ptr || !s_cuda_stream) return nullptr;
    return PyModule_Create(&module);
}
