// Python calls of the entry points that a training step makes once or more per EST, converted and made in
// native code.  A call of libes enqueues a launch (2.3 us of the runtime); ctypes added 0.35 to 1.1 us to it,
// a quarter of what a short BatchNorm layer costs, most of it per argument.
//
// A bound call takes plain ints, floats and None.  Whatever else ctypes accepts or refuses (other numbers,
// ctypes objects, keywords, defaults, too few arguments) goes to the Python function it stands for, `__wrapped__`.
// The interpreter lock is released around the call, as ctypes does.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <structmember.h>

#include <cstddef>
#include <cstdint>
#include <cstring>
#include <tuple>
#include <utility>

#include "es.h"

namespace {

struct Bound {
    PyObject_HEAD
    vectorcallfunc call;
    void* fn;
    PyObject* general;
};

// false: not a value that this file converts (no Python error is left)
bool unsigned_of(PyObject* o, uint64_t most, uint64_t& out)
{
    if (!PyLong_CheckExact(o)) return false;
    out = PyLong_AsUnsignedLongLong(o);
    if (out == (uint64_t)-1 && PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    return out <= most;
}
bool get(PyObject* o, uint64_t& out) { return unsigned_of(o, ~0ull, out); }
bool get(PyObject* o, uint32_t& out)
{
    uint64_t v = 0;
    if (!unsigned_of(o, 0xFFFFFFFFull, v)) return false;
    out = (uint32_t)v;
    return true;
}
template <class T>
bool get(PyObject* o, T*& out)
{
    uint64_t v = 0;
    if (o != Py_None && !unsigned_of(o, ~0ull, v)) return false;
    out = (T*)(uintptr_t)v;
    return true;
}
bool get(PyObject* o, double& out)
{
    if (!PyFloat_CheckExact(o)) return false;
    out = PyFloat_AS_DOUBLE(o);
    return true;
}
bool get(PyObject* o, float& out)
{
    double d = 0;
    if (!get(o, d)) return false;
    out = (float)d;
    return true;
}

template <class F>
struct Call;
template <class... A>
struct Call<int (*)(A...)> {
    template <size_t... I>
    static bool convert(PyObject* const* args, std::tuple<A...>& to, std::index_sequence<I...>)
    {
        return (get(args[I], std::get<I>(to)) && ...);
    }
    static PyObject* call(PyObject* self, PyObject* const* args, size_t nargsf, PyObject* names)
    {
        const Bound* b = reinterpret_cast<const Bound*>(self);
        std::tuple<A...> v;
        if ((names && PyTuple_GET_SIZE(names)) || PyVectorcall_NARGS(nargsf) != (Py_ssize_t)sizeof...(A) ||
            !convert(args, v, std::index_sequence_for<A...>{}))
            return PyObject_Vectorcall(b->general, args, PyVectorcall_NARGS(nargsf), names);
        int status = 0;
        auto fn = reinterpret_cast<int (*)(A...)>(b->fn);
        Py_BEGIN_ALLOW_THREADS
        status = std::apply(fn, v);
        Py_END_ALLOW_THREADS
        return PyLong_FromLong(status);
    }
};

const struct {
    const char* name;
    vectorcallfunc call;
} kCalls[] = {
#define ES_CALL(f) {#f, Call<decltype(&f)>::call}
    ES_CALL(es_ctx_restore),
    ES_CALL(es_ctx_save),
    ES_CALL(es_ctx_switch),
    ES_CALL(es_accumulate),
    ES_CALL(es_est_boundary),
    ES_CALL(es_stage_fence),
    ES_CALL(es_dropout_mask),
    ES_CALL(es_ring_order_reduce),
    ES_CALL(es_sgd_step),
    ES_CALL(es_reduce_sgd_step),
    ES_CALL(es_grad_sq_norm),
    ES_CALL(es_grad_sq_norm_static),
    ES_CALL(es_clip_sgd_step),
    ES_CALL(es_bn_batch_stats),
#undef ES_CALL
};

void bound_dealloc(PyObject* self)
{
    Py_DECREF(reinterpret_cast<Bound*>(self)->general);
    Py_TYPE(self)->tp_free(self);
}

// What the bound call does not have itself (its name, its documentation) is that of the function it stands for.
PyObject* bound_getattr(PyObject* self, PyObject* name)
{
    PyObject* general = reinterpret_cast<Bound*>(self)->general;
    const char* s = PyUnicode_AsUTF8(name);
    if (!s) return nullptr;
    if (!std::strcmp(s, "__wrapped__")) {
        Py_INCREF(general);
        return general;
    }
    if (!std::strcmp(s, "__class__") || !std::strcmp(s, "__call__")) return PyObject_GenericGetAttr(self, name);
    return PyObject_GetAttr(general, name);
}

PyTypeObject bound_type = {PyVarObject_HEAD_INIT(nullptr, 0)};

PyObject* bind(PyObject*, PyObject* args)
{
    const char* name;
    unsigned long long fn;
    PyObject* general;
    if (!PyArg_ParseTuple(args, "sKO", &name, &fn, &general)) return nullptr;
    for (const auto& c : kCalls) {
        if (std::strcmp(c.name, name) || !fn) continue;
        Bound* b = PyObject_New(Bound, &bound_type);
        if (!b) return nullptr;
        b->call = c.call;
        b->fn = (void*)(uintptr_t)fn;
        Py_INCREF(general);
        b->general = general;
        return reinterpret_cast<PyObject*>(b);
    }
    PyErr_SetString(PyExc_ValueError, name);
    return nullptr;
}

PyMethodDef methods[] = {{"bind", bind, METH_VARARGS, "bind(name, address, general): the native call of an entry point"},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pycall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pycall()
{
    bound_type.tp_name = "_pycall.Bound";
    bound_type.tp_basicsize = sizeof(Bound);
    bound_type.tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_VECTORCALL;
    bound_type.tp_vectorcall_offset = offsetof(Bound, call);
    bound_type.tp_call = PyVectorcall_Call;
    bound_type.tp_dealloc = bound_dealloc;
    bound_type.tp_getattro = bound_getattr;
    if (PyType_Ready(&bound_type) < 0) return nullptr;
    PyObject* m = PyModule_Create(&module);
    if (!m) return nullptr;
    constexpr Py_ssize_t n = sizeof(kCalls) / sizeof(kCalls[0]);
    PyObject* names = PyTuple_New(n);
    if (!names) { Py_DECREF(m); return nullptr; }
    for (Py_ssize_t i = 0; i < n; ++i) {
        PyObject* s = PyUnicode_FromString(kCalls[i].name);
        if (!s) { Py_DECREF(names); Py_DECREF(m); return nullptr; }
        PyTuple_SET_ITEM(names, i, s);
    }
    if (PyModule_AddObject(m, "NAMES", names) < 0) { Py_DECREF(names); Py_DECREF(m); return nullptr; }
    if (PyModule_AddStringConstant(m, "SOURCE_HASH", ES_PYCALL_HASH) < 0) { Py_DECREF(m); return nullptr; }
    return m;
}
