// The Python binding's hot calls, as an extension module: what it takes to hand a decode or recovery call to the library.
//
// ctypes takes 1 us to convert the arguments of a prepared call and 1.2 to 3.2 us to build the arrays of one named anew, where a launch takes 2.6 us and
// the kernels of a small call 3 to 6.  us of host time per call, ctypes / this: prepared, one tensor 3.7 / 2.75, three 3.75 / 2.8, 24 unlike ones 4.1 / 3.6;
// named anew, one tensor 5.1 / 3.0, three 5.2 / 2.9, 24 unlike ones 7.6 / 4.1; 24 addresses to a layer's handle 6.2 / 4.0; recovery 3.0 / 2.8.
//
// The functions come as addresses from the library that the binding has loaded.  Arguments of other types than the usual ones (lists or tuples
// of ints, objects with data_ptr) are left to the binding's ctypes path: a call answers None for them before it has done anything.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <structmember.h>

#include <cstddef>
#include <cstdint>

#include "zipmoe.h"

namespace {

constexpr Py_ssize_t kMost = 256;      // tensors of a call; longer ones are refused by the library

using DecodeFn = int (*)(const void *const *, const uint64_t *const *, const zm_tensor_info *, int, int, const int32_t *, int, void *const *, int, void *);
using LayerFn = int (*)(const zm_layer *, const int32_t *, int, void *const *, int, void *);
using RecoverFn = int (*)(const void *, const void *, size_t, void *, void *);

PyObject *data_ptr_name;

// An int as it is, of at most 64 bits.
bool plain(PyObject *o, uint64_t &v)
{
    if (!PyLong_CheckExact(o)) return false;
    int over = 0;
    const long long s = PyLong_AsLongLongAndOverflow(o, &over);
    if (!over) { v = static_cast<uint64_t>(s); return true; }
    if (over < 0) return false;
    v = PyLong_AsUnsignedLongLong(o);
    if (v == static_cast<uint64_t>(-1) && PyErr_Occurred()) { PyErr_Clear(); return false; }
    return true;
}

bool plain_int(PyObject *o, int &v)
{
    uint64_t u;
    if (!plain(o, u) || static_cast<int64_t>(u) != static_cast<int32_t>(u)) return false;
    v = static_cast<int>(static_cast<int64_t>(u));
    return true;
}

bool is_row(PyObject *o) { return PyList_CheckExact(o) || PyTuple_CheckExact(o); }

// Expert ids of a call; -1: left to the caller's other path.
Py_ssize_t read_ids(PyObject *o, int32_t *ids)
{
    if (!is_row(o)) return -1;
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(o);
    if (n > kMost) return -1;
    for (Py_ssize_t i = 0; i < n; ++i) {
        int v;
        if (!plain_int(PySequence_Fast_GET_ITEM(o, i), v)) return -1;
        ids[i] = v;
    }
    return n;
}

template <class F>
PyObject *status(F call)
{
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = call();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// ---- the arrays that describe a layer, and calls on it ----

struct Arrays {
    DecodeFn fn;
    const void *const *blobs;
    const uint64_t *const *tables;
    const zm_tensor_info *infos;
    int n_experts, per_expert;
};

struct Target {
    PyObject_HEAD
    Arrays a;
};

bool read_arrays(Arrays &a, unsigned long long fn, unsigned long long blobs, unsigned long long tables, unsigned long long infos)
{
    a.fn = reinterpret_cast<DecodeFn>(fn);
    a.blobs = reinterpret_cast<const void *const *>(blobs);
    a.tables = reinterpret_cast<const uint64_t *const *>(tables);
    a.infos = reinterpret_cast<const zm_tensor_info *>(infos);
    return fn != 0;
}

// Target(fn, blobs, tables, infos, n_experts, tensors_per_expert): addresses of zm_decode_experts_stores and of its arrays, which have to outlive it
PyObject *target_new(PyTypeObject *type, PyObject *args, PyObject *)
{
    unsigned long long fn, blobs, tables, infos;
    int n_experts, per_expert;
    if (!PyArg_ParseTuple(args, "KKKKii", &fn, &blobs, &tables, &infos, &n_experts, &per_expert)) return nullptr;
    Target *t = reinterpret_cast<Target *>(type->tp_alloc(type, 0));
    if (!t) return nullptr;
    if (!read_arrays(t->a, fn, blobs, tables, infos)) { Py_DECREF(t); PyErr_SetString(PyExc_ValueError, "no function"); return nullptr; }
    t->a.n_experts = n_experts;
    t->a.per_expert = per_expert;
    return reinterpret_cast<PyObject *>(t);
}

// decode(expert_ids, out_buffers, starts, stream, stores) -> status, or None
PyObject *target_decode(PyObject *self, PyObject *const *args, Py_ssize_t nargs)
{
    const Arrays &a = reinterpret_cast<Target *>(self)->a;
    int32_t ids[kMost];
    void *outs[kMost];
    uint64_t stream, offset[kMost];
    int stores;
    if (nargs != 5) Py_RETURN_NONE;
    PyObject *bufs = args[1], *starts = args[2];
    const Py_ssize_t n = read_ids(args[0], ids), per = a.per_expert;
    if (n < 0 || per < 1 || per > kMost || n * per > kMost || !is_row(bufs) || !PyList_CheckExact(starts) || PyList_GET_SIZE(starts) < per || !plain(args[3], stream) ||
        !plain_int(args[4], stores)) Py_RETURN_NONE;
    const Py_ssize_t n_bufs = PySequence_Fast_GET_SIZE(bufs);
    if (n_bufs > n) Py_RETURN_NONE;
    for (Py_ssize_t m = 0; m < per; ++m)
        if (!plain(PyList_GET_ITEM(starts, m), offset[m])) Py_RETURN_NONE;
    for (Py_ssize_t j = 0; j < n; ++j) {
        uint64_t base = 0;
        if (j < n_bufs) {
            if (j >= PySequence_Fast_GET_SIZE(bufs)) Py_RETURN_NONE;          // a data_ptr that shortens the list
            PyObject *p = PyObject_CallMethodNoArgs(PySequence_Fast_GET_ITEM(bufs, j), data_ptr_name);
            if (!p) return nullptr;
            const bool ok = plain(p, base);
            Py_DECREF(p);
            if (!ok) Py_RETURN_NONE;
        }
        for (Py_ssize_t m = 0; m < per; ++m) outs[j * per + m] = reinterpret_cast<void *>(j < n_bufs ? base + 2 * offset[m] : 0);
    }
    return status([&] { return a.fn(a.blobs, a.tables, a.infos, a.n_experts, a.per_expert, ids, static_cast<int>(n), outs, stores, reinterpret_cast<void *>(stream)); });
}

PyMethodDef target_methods[] = {{"decode", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(target_decode)), METH_FASTCALL, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyTypeObject target_type = {PyVarObject_HEAD_INIT(nullptr, 0)};

// ---- a call whose arrays are there ----

struct Prepared {
    PyObject_HEAD
    vectorcallfunc vectorcall;
    Arrays a;
    const int32_t *ids;
    void *const *outs;
    int n, stores;
    PyObject *keepalive, *owner, *check, *dict;
};

// call(stream=0)
PyObject *prepared_call(PyObject *self, PyObject *const *args, size_t nargsf, PyObject *kwnames)
{
    Prepared *p = reinterpret_cast<Prepared *>(self);
    const Py_ssize_t given = PyVectorcall_NARGS(nargsf), named = kwnames ? PyTuple_GET_SIZE(kwnames) : 0;
    if (given + named > 1 || (named && PyUnicode_CompareWithASCIIString(PyTuple_GET_ITEM(kwnames, 0), "stream") != 0)) {
        PyErr_SetString(PyExc_TypeError, "call() takes one optional argument: stream");
        return nullptr;
    }
    uint64_t stream = 0;
    if (given + named && args[0] != Py_None && !plain(args[0], stream)) {
        if (!PyLong_Check(args[0])) {
            PyErr_SetString(PyExc_TypeError, "cannot be converted to pointer");
            return nullptr;
        }
        stream = PyLong_AsUnsignedLongLongMask(args[0]);
        if (stream == static_cast<uint64_t>(-1) && PyErr_Occurred()) return nullptr;
    }
    int rc;
    Py_INCREF(self);
    Py_BEGIN_ALLOW_THREADS
    rc = p->a.fn(p->a.blobs, p->a.tables, p->a.infos, p->a.n_experts, p->a.per_expert, p->ids, p->n, p->outs, p->stores, reinterpret_cast<void *>(stream));
    Py_END_ALLOW_THREADS
    PyObject *res = Py_None;
    if (rc == ZM_OK) Py_INCREF(res);
    else res = PyObject_CallFunction(p->check, "i", rc);
    Py_DECREF(self);
    return res;
}

// Prepared(fn, blobs, tables, infos, n_experts, tensors_per_expert, ids, n_selected, outs, stores, keepalive, owner, check): keepalive and owner hold what
// the addresses point at; check(status) is called when the status is not ZM_OK, and raises
PyObject *prepared_new(PyTypeObject *type, PyObject *args, PyObject *)
{
    unsigned long long fn, blobs, tables, infos, ids, outs;
    int n_experts, per_expert, n, stores;
    PyObject *keepalive, *owner, *check;
    if (!PyArg_ParseTuple(args, "KKKKiiKiKiOOO", &fn, &blobs, &tables, &infos, &n_experts, &per_expert, &ids, &n, &outs, &stores, &keepalive, &owner, &check)) return nullptr;
    Prepared *p = reinterpret_cast<Prepared *>(type->tp_alloc(type, 0));
    if (!p) return nullptr;
    p->vectorcall = prepared_call;
    p->ids = reinterpret_cast<const int32_t *>(ids);
    p->outs = reinterpret_cast<void *const *>(outs);
    p->n = n;
    p->stores = stores;
    Py_INCREF(p->keepalive = keepalive);
    Py_INCREF(p->owner = owner);
    Py_INCREF(p->check = check);
    p->dict = nullptr;
    if (!read_arrays(p->a, fn, blobs, tables, infos)) { Py_DECREF(p); PyErr_SetString(PyExc_ValueError, "no function"); return nullptr; }
    p->a.n_experts = n_experts;
    p->a.per_expert = per_expert;
    return reinterpret_cast<PyObject *>(p);
}

int prepared_traverse(PyObject *self, visitproc visit, void *arg)
{
    Prepared *p = reinterpret_cast<Prepared *>(self);
    Py_VISIT(p->keepalive);
    Py_VISIT(p->owner);
    Py_VISIT(p->check);
    Py_VISIT(p->dict);
    return 0;
}
int prepared_clear(PyObject *self)
{
    Prepared *p = reinterpret_cast<Prepared *>(self);
    // what the addresses point at goes: a call from a finalizer that comes after finds nothing selected
    p->n = 0;
    Py_CLEAR(p->keepalive);
    Py_CLEAR(p->owner);
    Py_CLEAR(p->check);
    Py_CLEAR(p->dict);
    return 0;
}
void prepared_dealloc(PyObject *self)
{
    PyObject_GC_UnTrack(self);
    prepared_clear(self);
    Py_TYPE(self)->tp_free(self);
}

PyMemberDef prepared_members[] = {{"keepalive", T_OBJECT, offsetof(Prepared, keepalive), READONLY, nullptr}, {nullptr, 0, 0, 0, nullptr}};
PyGetSetDef prepared_getset[] = {{"__dict__", PyObject_GenericGetDict, PyObject_GenericSetDict, nullptr, nullptr}, {nullptr, nullptr, nullptr, nullptr, nullptr}};
PyTypeObject prepared_type = {PyVarObject_HEAD_INIT(nullptr, 0)};

// ---- functions ----

// layer_decode(fn, handle, expert_ids, out_ptrs, stream, stores) -> status, or None
PyObject *layer_decode(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    int32_t ids[kMost];
    void *outs[kMost];
    uint64_t fn, handle, stream;
    int stores;
    if (nargs != 6 || !plain(args[0], fn) || !plain(args[1], handle) || !is_row(args[3]) || !plain(args[4], stream) || !plain_int(args[5], stores)) Py_RETURN_NONE;
    const Py_ssize_t n = read_ids(args[2], ids), n_outs = PySequence_Fast_GET_SIZE(args[3]);
    if (n < 0 || n_outs > kMost) Py_RETURN_NONE;
    for (Py_ssize_t i = 0; i < n_outs; ++i) {
        uint64_t p;
        if (!plain(PySequence_Fast_GET_ITEM(args[3], i), p)) Py_RETURN_NONE;
        outs[i] = reinterpret_cast<void *>(p);
    }
    for (Py_ssize_t i = n_outs; i < kMost; ++i) outs[i] = nullptr;         // a missing address is refused by the library
    return status([&] { return reinterpret_cast<LayerFn>(fn)(reinterpret_cast<const zm_layer *>(handle), ids, static_cast<int>(n), outs, stores, reinterpret_cast<void *>(stream)); });
}

// recover(fn, exponents, sign_mantissa, n_values, out, stream) -> status, or None
PyObject *recover(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    uint64_t v[6];
    if (nargs != 6) Py_RETURN_NONE;
    for (int i = 0; i < 6; ++i)
        if (!plain(args[i], v[i])) Py_RETURN_NONE;
    return status([&] {
        return reinterpret_cast<RecoverFn>(v[0])(reinterpret_cast<const void *>(v[1]), reinterpret_cast<const void *>(v[2]), v[3], reinterpret_cast<void *>(v[4]), reinterpret_cast<void *>(v[5]));
    });
}

PyMethodDef functions[] = {{"layer_decode", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(layer_decode)), METH_FASTCALL, nullptr},
                           {"recover", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(recover)), METH_FASTCALL, nullptr},
                           {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, functions, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native()
{
    target_type.tp_name = "paper_2601_21198_amd._native.Target";
    target_type.tp_basicsize = sizeof(Target);
    target_type.tp_flags = Py_TPFLAGS_DEFAULT;
    target_type.tp_new = target_new;
    target_type.tp_methods = target_methods;
    prepared_type.tp_name = "paper_2601_21198_amd._native.Prepared";
    prepared_type.tp_basicsize = sizeof(Prepared);
    prepared_type.tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_GC | Py_TPFLAGS_HAVE_VECTORCALL;
    prepared_type.tp_new = prepared_new;
    prepared_type.tp_call = PyVectorcall_Call;
    prepared_type.tp_vectorcall_offset = offsetof(Prepared, vectorcall);
    prepared_type.tp_dictoffset = offsetof(Prepared, dict);
    prepared_type.tp_members = prepared_members;
    prepared_type.tp_getset = prepared_getset;
    prepared_type.tp_traverse = prepared_traverse;
    prepared_type.tp_clear = prepared_clear;
    prepared_type.tp_dealloc = prepared_dealloc;
    if (PyType_Ready(&target_type) < 0 || PyType_Ready(&prepared_type) < 0) return nullptr;
    data_ptr_name = PyUnicode_InternFromString("data_ptr");
    PyObject *m = PyModule_Create(&module);
    if (!m || !data_ptr_name) return nullptr;
    Py_INCREF(&target_type);
    Py_INCREF(&prepared_type);
    if (PyModule_AddObject(m, "Target", reinterpret_cast<PyObject *>(&target_type)) < 0 || PyModule_AddObject(m, "Prepared", reinterpret_cast<PyObject *>(&prepared_type)) < 0) return nullptr;
    return m;
}
