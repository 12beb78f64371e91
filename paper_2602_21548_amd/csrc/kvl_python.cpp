// The per-layer calls of the Python binding, from Python objects to the C ABI in one step (module _native).
//
// A layer of a few MB takes its kernels 3 us each, and ctypes with its argument objects took 5 us a call on the host.
// Here a call reads the tensors' addresses and sizes by the same attributes that binding.py reads, and calls the same
// entry point of the same library.  Whatever is not plainly in order (an argument of another type, a tensor that is not
// contiguous, a pool or a buffer too small, a plan destroyed) is left to binding.py, which says what is wrong with it or
// takes it: the functions return 1 for that, else what the library returned.  A hop of 4.6 MB 17.3 -> 8.3 us (6.3 of kernels;
// the same through the C ABI with arguments made before 7.9); the requests of a batch of 64 for kvl_plan 120 -> 2.3.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <structmember.h>

#include <cstdint>

#include "kvl.h"

namespace {

constexpr long kNotTaken = 1;

// What binding.py's Plan objects add to Python's own: the handle and what is asked of a pool on every call.
struct PlanObject {
    PyObject_HEAD
    void *handle;                              // null: destroyed, or not set
    Py_ssize_t planes;
    unsigned long long bytes[KVL_MAX_PLANES];
    Py_ssize_t dst_planes;                     // of paired plans
    unsigned long long dst_bytes[KVL_MAX_PLANES];
};

struct Library {
    decltype(&kvl_pack_layer) pack;
    decltype(&kvl_unpack_layer) unpack;
    decltype(&kvl_move_layer) move;
    decltype(&kvl_fullblocks_to_pool_layer) to_pool;
    decltype(&kvl_pool_to_fullblocks_layer) to_blocks;
} g_lib;
PyObject *g_tensor_type, *g_array_type, *g_raw_stream, *g_get_device, *g_is_initialized;
bool g_initialized;             // this process has a device context (a forked child starts anew)
PyObject *s_is_cuda, *s_is_contiguous, *s_is_pinned, *s_data_ptr, *s_nbytes, *s_cuda_stream;

PyTypeObject *plan_type();

// Python's attributes and methods by name; false (with no exception left) if anything is unlike what is expected.
bool get_true(PyObject *o, PyObject *name, bool *value) {
    PyObject *r = PyObject_GetAttr(o, name);
    if (r != Py_True && r != Py_False) {
        Py_XDECREF(r);
        PyErr_Clear();
        return false;
    }
    *value = r == Py_True;
    Py_DECREF(r);
    return true;
}
bool call_true(PyObject *o, PyObject *name) {
    PyObject *args[1] = {o};
    PyObject *r = PyObject_VectorcallMethod(name, args, 1 | PY_VECTORCALL_ARGUMENTS_OFFSET, nullptr);
    if (!r) PyErr_Clear();
    const bool yes = r == Py_True;
    Py_XDECREF(r);
    return yes;
}
bool number(PyObject *r, unsigned long long *value) {       // (takes the reference)
    if (!r || !PyLong_Check(r)) {
        Py_XDECREF(r);
        PyErr_Clear();
        return false;
    }
    *value = PyLong_AsUnsignedLongLong(r);
    Py_DECREF(r);
    if (*value == (unsigned long long)-1 && PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    return true;
}

struct Buffer {
    void *ptr;
    unsigned long long bytes;
};
// A contiguous tensor on the device or, where `host` is given, in pinned memory.
bool buffer(PyObject *t, bool host, Buffer *out) {
    if ((PyObject *)Py_TYPE(t) != g_tensor_type) return false;
    bool cuda;
    if (!get_true(t, s_is_cuda, &cuda) || (!cuda && !(host && call_true(t, s_is_pinned)))) return false;
    if (!call_true(t, s_is_contiguous)) return false;
    unsigned long long p;
    PyObject *args[1] = {t};
    if (!number(PyObject_VectorcallMethod(s_data_ptr, args, 1 | PY_VECTORCALL_ARGUMENTS_OFFSET, nullptr), &p)) return false;
    if (!number(PyObject_GetAttr(t, s_nbytes), &out->bytes)) return false;
    out->ptr = (void *)(uintptr_t)p;
    return true;
}

bool pool(PyObject *planes, Py_ssize_t n, const unsigned long long *need, void **out) {
    const bool list = PyList_CheckExact(planes);
    if (!list && !PyTuple_CheckExact(planes)) return false;
    if (n == 0 || (list ? PyList_GET_SIZE(planes) : PyTuple_GET_SIZE(planes)) != n) return false;
    for (Py_ssize_t p = 0; p < n; ++p) {
        // (the attributes run Python code at most for exotic tensors, but a list could be changed by it)
        if (list && PyList_GET_SIZE(planes) != n) return false;
        PyObject *t = list ? PyList_GET_ITEM(planes, p) : PyTuple_GET_ITEM(planes, p);
        Py_INCREF(t);
        Buffer b;
        const bool ok = buffer(t, false, &b) && b.bytes >= need[p];
        Py_DECREF(t);
        if (!ok) return false;
        out[p] = b.ptr;
    }
    return true;
}

bool stream(PyObject *s, void **out) {
    unsigned long long h;
    if (s == Py_None) {
        if (!g_initialized) {
            PyObject *r = PyObject_CallNoArgs(g_is_initialized);
            if (!r) PyErr_Clear();
            g_initialized = r == Py_True;
            Py_XDECREF(r);
            if (!g_initialized) return false;
        }
        PyObject *device = PyObject_CallNoArgs(g_get_device);
        if (!device) {
            PyErr_Clear();
            return false;
        }
        PyObject *r = PyObject_CallOneArg(g_raw_stream, device);
        Py_DECREF(device);
        if (!number(r, &h)) return false;
    } else if (PyLong_Check(s)) {
        Py_INCREF(s);
        if (!number(s, &h)) return false;
    } else if (!number(PyObject_GetAttr(s, s_cuda_stream), &h)) {
        return false;
    }
    *out = (void *)(uintptr_t)h;
    return true;
}

PlanObject *plan_of(PyObject *o) {
    if (!PyObject_TypeCheck(o, plan_type())) return nullptr;
    PlanObject *p = (PlanObject *)o;
    return p->handle ? p : nullptr;
}

// (As ctypes does, the interpreter goes on meanwhile.)
#define KVL_CALL(expr)              \
    do {                            \
        int rc;                     \
        Py_BEGIN_ALLOW_THREADS      \
        rc = (expr);                \
        Py_END_ALLOW_THREADS        \
        return PyLong_FromLong(rc); \
    } while (0)
#define KVL_NOT_TAKEN return PyLong_FromLong(kNotTaken)

PyObject *pack_layer(PyObject *, PyObject *const *a, Py_ssize_t n) {        // plan, pool planes, xfer, stream
    PlanObject *plan = n == 4 ? plan_of(a[0]) : nullptr;
    void *planes[KVL_MAX_PLANES], *s;
    Buffer x;
    if (!plan || !pool(a[1], plan->planes, plan->bytes, planes) || !buffer(a[2], true, &x) || !stream(a[3], &s)) KVL_NOT_TAKEN;
    void *handle = plan->handle;
    KVL_CALL(g_lib.pack((const kvl_plan_t *)handle, planes, x.ptr, x.bytes, s));
}

PyObject *unpack_layer(PyObject *, PyObject *const *a, Py_ssize_t n) {      // plan, xfer, pool planes, stream
    PlanObject *plan = n == 4 ? plan_of(a[0]) : nullptr;
    void *planes[KVL_MAX_PLANES], *s;
    Buffer x;
    if (!plan || !pool(a[2], plan->planes, plan->bytes, planes) || !buffer(a[1], true, &x) || !stream(a[3], &s)) KVL_NOT_TAKEN;
    void *handle = plan->handle;
    KVL_CALL(g_lib.unpack((const kvl_plan_t *)handle, x.ptr, x.bytes, planes, s));
}

PyObject *move_layer(PyObject *, PyObject *const *a, Py_ssize_t n) {        // plan, source planes, destination planes, stream
    PlanObject *plan = n == 4 ? plan_of(a[0]) : nullptr;
    void *src[KVL_MAX_PLANES], *dst[KVL_MAX_PLANES], *s;
    if (!plan || !pool(a[1], plan->planes, plan->bytes, src) || !pool(a[2], plan->dst_planes, plan->dst_bytes, dst) || !stream(a[3], &s))
        KVL_NOT_TAKEN;
    void *handle = plan->handle;
    KVL_CALL(g_lib.move((const kvl_plan_t *)handle, src, dst, s));
}

bool layer_of(PyObject *o, uint32_t *layer) {
    unsigned long long v;
    if (!PyLong_CheckExact(o)) return false;
    Py_INCREF(o);
    if (!number(o, &v) || v > UINT32_MAX) return false;
    *layer = (uint32_t)v;
    return true;
}

PyObject *fullblocks_to_pool_layer(PyObject *, PyObject *const *a, Py_ssize_t n) {      // plan, blocks, layer, planes, stream
    PlanObject *plan = n == 5 ? plan_of(a[0]) : nullptr;
    void *planes[KVL_MAX_PLANES], *s;
    Buffer b;
    uint32_t layer;
    if (!plan || !pool(a[3], plan->planes, plan->bytes, planes) || !buffer(a[1], true, &b) || !layer_of(a[2], &layer) || !stream(a[4], &s))
        KVL_NOT_TAKEN;
    void *handle = plan->handle;
    KVL_CALL(g_lib.to_pool((const kvl_plan_t *)handle, b.ptr, b.bytes, layer, planes, s));
}

PyObject *pool_to_fullblocks_layer(PyObject *, PyObject *const *a, Py_ssize_t n) {      // plan, planes, layer, blocks, stream
    PlanObject *plan = n == 5 ? plan_of(a[0]) : nullptr;
    void *planes[KVL_MAX_PLANES], *s;
    Buffer b;
    uint32_t layer;
    if (!plan || !pool(a[1], plan->planes, plan->bytes, planes) || !buffer(a[3], true, &b) || !layer_of(a[2], &layer) || !stream(a[4], &s))
        KVL_NOT_TAKEN;
    void *handle = plan->handle;
    KVL_CALL(g_lib.to_blocks((const kvl_plan_t *)handle, planes, layer, b.ptr, b.bytes, s));
}

// requests(hit, app, tables, out): a batch's kvl_request_t into `out`, from contiguous uint32 arrays and a list of contiguous
// int32 tables, all of them NumPy's.  False: not all of them are that.
bool array_of(PyObject *o, const char *formats, Py_buffer *view) {
    if (PyObject_GetBuffer(o, view, PyBUF_C_CONTIGUOUS | PyBUF_FORMAT) != 0) {
        PyErr_Clear();
        return false;
    }
    const char *f = view->format;
    if (view->itemsize == 4 && f && f[0] && !f[1] && (f[0] == formats[0] || f[0] == formats[1])) return true;
    PyBuffer_Release(view);
    return false;
}
PyObject *requests(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (n != 4 || !PyList_CheckExact(a[2])) Py_RETURN_FALSE;
    const Py_ssize_t count = PyList_GET_SIZE(a[2]);
    Py_buffer hit, app, out;
    if (!array_of(a[0], "IL", &hit)) Py_RETURN_FALSE;
    if (!array_of(a[1], "IL", &app)) {
        PyBuffer_Release(&hit);
        Py_RETURN_FALSE;
    }
    bool ok = hit.len / 4 == count && app.len / 4 == count;
    if (ok && PyObject_GetBuffer(a[3], &out, PyBUF_WRITABLE) != 0) {
        PyErr_Clear();
        ok = false;
    }
    if (ok) {
        ok = out.len >= (Py_ssize_t)sizeof(kvl_request_t) * count;
        kvl_request_t *r = (kvl_request_t *)out.buf;
        for (Py_ssize_t k = 0; k < count && ok; ++k) {
            Py_buffer t;
            PyObject *table = PyList_GET_ITEM(a[2], k);
            ok = (PyObject *)Py_TYPE(table) == g_array_type && array_of(table, "il", &t);
            if (!ok) break;
            ok = t.len / 4 <= (Py_ssize_t)UINT32_MAX;
            r[k].hit_tokens = ((const uint32_t *)hit.buf)[k];
            r[k].append_tokens = ((const uint32_t *)app.buf)[k];
            r[k].n_blocks = (uint32_t)(t.len / 4);
            r[k].block_table = t.len ? (const int32_t *)t.buf : nullptr;    // (the caller's list keeps the table)
            PyBuffer_Release(&t);
        }
        PyBuffer_Release(&out);
    }
    PyBuffer_Release(&hit);
    PyBuffer_Release(&app);
    return PyBool_FromLong(ok);
}

// setup(torch.Tensor, numpy.ndarray, torch's three stream functions, the addresses of the library's five entry points)
PyObject *setup(PyObject *, PyObject *args) {
    PyObject *type, *array, *raw, *device, *initialized;
    unsigned long long f[5];
    if (!PyArg_ParseTuple(args, "OOOOOKKKKK", &type, &array, &raw, &device, &initialized, &f[0], &f[1], &f[2], &f[3], &f[4])) return nullptr;
    Py_INCREF(type);
    Py_INCREF(array);
    Py_INCREF(raw);
    Py_INCREF(device);
    Py_INCREF(initialized);
    g_tensor_type = type;
    g_array_type = array;
    g_raw_stream = raw;
    g_get_device = device;
    g_is_initialized = initialized;
    g_lib.pack = (decltype(g_lib.pack))(uintptr_t)f[0];
    g_lib.unpack = (decltype(g_lib.unpack))(uintptr_t)f[1];
    g_lib.move = (decltype(g_lib.move))(uintptr_t)f[2];
    g_lib.to_pool = (decltype(g_lib.to_pool))(uintptr_t)f[3];
    g_lib.to_blocks = (decltype(g_lib.to_blocks))(uintptr_t)f[4];
    Py_RETURN_NONE;
}

PyObject *forked(PyObject *, PyObject *) {
    g_initialized = false;
    Py_RETURN_NONE;
}

PyObject *plan_set(PyObject *self, PyObject *args) {        // _set(handle, bytes of the pool's planes)
    PlanObject *p = (PlanObject *)self;
    unsigned long long handle, bytes[KVL_MAX_PLANES] = {};
    PyObject *t;
    if (!PyArg_ParseTuple(args, "KO!", &handle, &PyTuple_Type, &t)) return nullptr;
    const Py_ssize_t n = PyTuple_GET_SIZE(t);
    if (n > KVL_MAX_PLANES) {
        PyErr_SetString(PyExc_ValueError, "too many planes");
        return nullptr;
    }
    for (Py_ssize_t k = 0; k < n; ++k) {
        bytes[k] = PyLong_AsUnsignedLongLong(PyTuple_GET_ITEM(t, k));
        if (PyErr_Occurred()) return nullptr;
    }
    p->handle = (void *)(uintptr_t)handle;
    p->planes = n;
    for (Py_ssize_t k = 0; k < n; ++k) p->bytes[k] = bytes[k];
    Py_RETURN_NONE;
}
PyObject *plan_set_dst(PyObject *self, PyObject *t) {
    PlanObject *p = (PlanObject *)self;
    if (!PyTuple_CheckExact(t) || PyTuple_GET_SIZE(t) > KVL_MAX_PLANES) {
        PyErr_SetString(PyExc_TypeError, "need a tuple of plane sizes");
        return nullptr;
    }
    p->dst_planes = 0;
    for (Py_ssize_t k = 0; k < PyTuple_GET_SIZE(t); ++k) {
        p->dst_bytes[k] = PyLong_AsUnsignedLongLong(PyTuple_GET_ITEM(t, k));
        if (PyErr_Occurred()) return nullptr;
    }
    p->dst_planes = PyTuple_GET_SIZE(t);
    Py_RETURN_NONE;
}
PyObject *plan_clear(PyObject *self, PyObject *) {
    ((PlanObject *)self)->handle = nullptr;
    Py_RETURN_NONE;
}

PyMethodDef plan_methods[] = {
    {"_set", plan_set, METH_VARARGS, nullptr},
    {"_set_dst", plan_set_dst, METH_O, nullptr},
    {"_clear", plan_clear, METH_NOARGS, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

PyTypeObject g_plan_type = {PyVarObject_HEAD_INIT(nullptr, 0)};
PyTypeObject *plan_type() { return &g_plan_type; }

PyMethodDef module_methods[] = {
    {"pack_layer", (PyCFunction)(void (*)(void))pack_layer, METH_FASTCALL, nullptr},
    {"unpack_layer", (PyCFunction)(void (*)(void))unpack_layer, METH_FASTCALL, nullptr},
    {"move_layer", (PyCFunction)(void (*)(void))move_layer, METH_FASTCALL, nullptr},
    {"fullblocks_to_pool_layer", (PyCFunction)(void (*)(void))fullblocks_to_pool_layer, METH_FASTCALL, nullptr},
    {"pool_to_fullblocks_layer", (PyCFunction)(void (*)(void))pool_to_fullblocks_layer, METH_FASTCALL, nullptr},
    {"requests", (PyCFunction)(void (*)(void))requests, METH_FASTCALL, nullptr},
    {"setup", setup, METH_VARARGS, nullptr},
    {"forked", forked, METH_NOARGS, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

// (found in the file by build.py, which takes no module built from other sources: the calls above go by raw addresses)
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", "The per-layer calls of the binding (" KVL_NATIVE_KEY ")", -1, module_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) {
    const char *names[] = {"is_cuda", "is_contiguous", "is_pinned", "data_ptr", "nbytes", "cuda_stream"};
    PyObject **where[] = {&s_is_cuda, &s_is_contiguous, &s_is_pinned, &s_data_ptr, &s_nbytes, &s_cuda_stream};
    for (int i = 0; i < 6; ++i)
        if (!(*where[i] = PyUnicode_InternFromString(names[i]))) return nullptr;
    g_plan_type.tp_name = "paper_2602_21548_amd._native.PlanBase";
    g_plan_type.tp_basicsize = sizeof(PlanObject);
    g_plan_type.tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_BASETYPE;
    g_plan_type.tp_new = PyType_GenericNew;
    g_plan_type.tp_methods = plan_methods;
    if (PyType_Ready(&g_plan_type) < 0) return nullptr;
    PyObject *m = PyModule_Create(&module);
    if (!m) return nullptr;
    Py_INCREF(&g_plan_type);
    if (PyModule_AddObject(m, "PlanBase", (PyObject *)&g_plan_type) < 0) {
        Py_DECREF(&g_plan_type);
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
