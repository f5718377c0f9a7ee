// Python calls of the C ABI without an interpreter in between: one callable object per entry point
// that turns its arguments into the C ones and calls.
//
// A layer while generating is two or three calls of a few microseconds of GPU time each, and HIP
// takes 2.4 us of the host for a launch: what the host adds around it decides whether the GPU waits.
// Through ctypes a call cost 6.7 us, 2.7 of them torch.cuda.current_stream() building a Python
// object and 1.6 the marshalling; through here it costs 2.9.
//
// The objects know nothing of a library file: connect() hands them the addresses of the
// entry points of the one that binding.py loaded.  Otherwise they are to a program what a function of binding.py is:
// they take attributes (binding.py gives them name, module, documentation and signature), weak references, pickle and
// copy by name and bind to an instance.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <stddef.h>

#include <type_traits>
#include <utility>

#include "../../include/qtip.h"

namespace {

constexpr int MAX_ARGS = 20;
enum Kind : char { POINTER, INTEGER, STREAM };

PyObject *g_address, *g_stream, *g_failed;         // binding.py: slow forms of an address and a stream; raise
PyObject *g_current_device, *g_raw_stream;         // torch: current device, its current stream as an integer
PyObject *g_load;                                  // binding.py: load the library and connect()
PyObject *s_data_ptr;

struct Entry {
    PyObject_HEAD
    vectorcallfunc call;
    const char *name;
    void *function;  // null until connect()
    int (*invoke)(void *function, const unsigned long long *args);
    int count, required;
    Kind kind[MAX_ARGS];
    PyObject *keyword[MAX_ARGS];
    PyObject *dict, *weak_references;
};

bool as_integer(PyObject *o, unsigned long long &out) {
    if (PyLong_Check(o)) {
        out = PyLong_AsUnsignedLongLongMask(o);
        return !(out == (unsigned long long)-1 && PyErr_Occurred());
    }
    PyObject *index = PyNumber_Index(o);
    if (!index) return false;
    out = PyLong_AsUnsignedLongLongMask(index);
    Py_DECREF(index);
    return !(out == (unsigned long long)-1 && PyErr_Occurred());
}
// takes the reference
bool take_integer(PyObject *o, unsigned long long &out) {
    if (!o) return false;
    if (o == Py_None) {
        out = 0;
        Py_DECREF(o);
        return true;
    }
    const bool ok = as_integer(o, out);
    Py_DECREF(o);
    return ok;
}

bool as_pointer(PyObject *o, unsigned long long &out) {
    if (o == Py_None) {
        out = 0;
        return true;
    }
    if (PyLong_Check(o)) return as_integer(o, out);
    PyObject *p = PyObject_CallMethodNoArgs(o, s_data_ptr);  // a torch tensor
    if (!p) {
        if (!PyErr_ExceptionMatches(PyExc_AttributeError)) return false;
        PyErr_Clear();
        p = PyObject_CallOneArg(g_address, o);
    }
    return take_integer(p, out);
}

bool as_stream(PyObject *o, unsigned long long &out) {
    if (!o || o == Py_None) {
        if (g_raw_stream) {
            PyObject *device = PyObject_CallNoArgs(g_current_device);
            if (!device) return false;
            PyObject *p = PyObject_CallOneArg(g_raw_stream, device);
            Py_DECREF(device);
            return take_integer(p, out);
        }
        return take_integer(PyObject_CallOneArg(g_stream, Py_None), out);
    }
    if (PyLong_Check(o)) return as_integer(o, out);
    return take_integer(PyObject_CallOneArg(g_stream, o), out);
}

PyObject *entry_call(PyObject *self, PyObject *const *args, size_t nargsf, PyObject *kwnames) {
    Entry *e = reinterpret_cast<Entry *>(self);
    const Py_ssize_t npos = PyVectorcall_NARGS(nargsf);
    PyObject *given[MAX_ARGS] = {};
    if (npos > e->count)
        return PyErr_Format(PyExc_TypeError, "%s() takes at most %d arguments (%zd given)", e->name, e->count, npos);
    for (Py_ssize_t i = 0; i < npos; i++) given[i] = args[i];
    const Py_ssize_t nkw = kwnames ? PyTuple_GET_SIZE(kwnames) : 0;
    for (Py_ssize_t k = 0; k < nkw; k++) {
        PyObject *key = PyTuple_GET_ITEM(kwnames, k);
        int at = -1;
        for (int i = 0; i < e->count && at < 0; i++)
            if (key == e->keyword[i]) at = i;
        for (int i = 0; i < e->count && at < 0; i++) {
            const int same = PyObject_RichCompareBool(key, e->keyword[i], Py_EQ);
            if (same < 0) return nullptr;
            if (same) at = i;
        }
        if (at < 0) return PyErr_Format(PyExc_TypeError, "%s() got an unexpected keyword argument '%U'", e->name, key);
        if (given[at]) return PyErr_Format(PyExc_TypeError, "%s() got multiple values for argument '%U'", e->name, key);
        given[at] = args[npos + k];
    }
    if (!e->function) {
        PyObject *r = PyObject_CallNoArgs(g_load);
        if (!r) return nullptr;
        Py_DECREF(r);
        if (!e->function) return PyErr_Format(PyExc_RuntimeError, "%s is not connected to a library", e->name);
    }
    unsigned long long value[MAX_ARGS];
    for (int i = 0; i < e->count; i++) {
        if (!given[i] && i < e->required)
            return PyErr_Format(PyExc_TypeError, "%s() missing required argument '%U'", e->name, e->keyword[i]);
        bool ok;
        if (e->kind[i] == STREAM) ok = as_stream(given[i], value[i]);
        else if (e->kind[i] == INTEGER) ok = as_integer(given[i], value[i]);
        else ok = as_pointer(given[i] ? given[i] : Py_None, value[i]);
        if (!ok) return nullptr;
    }
    int rc;
    Py_BEGIN_ALLOW_THREADS  // (a launch waits where the stream's queue is full)
    rc = e->invoke(e->function, value);
    Py_END_ALLOW_THREADS
    if (rc != 0) return PyObject_CallFunction(g_failed, "i", rc);
    return PyLong_FromLong(0);
}

void entry_dealloc(PyObject *self) {
    Entry *e = reinterpret_cast<Entry *>(self);
    PyObject_GC_UnTrack(self);
    if (e->weak_references) PyObject_ClearWeakRefs(self);
    Py_XDECREF(e->dict);
    for (int i = 0; i < e->count; i++) Py_XDECREF(e->keyword[i]);
    Py_TYPE(self)->tp_free(self);
}
int entry_traverse(PyObject *self, visitproc visit, void *arg) {
    Py_VISIT(reinterpret_cast<Entry *>(self)->dict);
    return 0;
}
int entry_clear(PyObject *self) {
    Py_CLEAR(reinterpret_cast<Entry *>(self)->dict);
    return 0;
}
PyObject *entry_repr(PyObject *self) {
    return PyUnicode_FromFormat("<entry point %s>", reinterpret_cast<Entry *>(self)->name);
}
PyObject *entry_get(PyObject *self, PyObject *instance, PyObject *) {
    if (instance && instance != Py_None) return PyMethod_New(self, instance);
    Py_INCREF(self);
    return self;
}
// (a name: pickle and copy look it up in __module__)
PyObject *entry_reduce(PyObject *self, PyObject *) {
    return PyUnicode_FromString(reinterpret_cast<Entry *>(self)->name);
}
PyMethodDef entry_methods[] = {{"__reduce__", entry_reduce, METH_NOARGS, nullptr}, {}};
PyGetSetDef entry_attributes[] = {{"__dict__", PyObject_GenericGetDict, PyObject_GenericSetDict, nullptr, nullptr}, {}};

PyTypeObject EntryType = [] {
    PyTypeObject t = {PyVarObject_HEAD_INIT(nullptr, 0)};
    t.tp_name = "paper_2406_11235_amd._call.Entry";
    t.tp_basicsize = sizeof(Entry);
    t.tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_VECTORCALL | Py_TPFLAGS_HAVE_GC;
    t.tp_vectorcall_offset = offsetof(Entry, call);
    t.tp_call = PyVectorcall_Call;
    t.tp_dealloc = entry_dealloc;
    t.tp_repr = entry_repr;
    t.tp_traverse = entry_traverse;
    t.tp_clear = entry_clear;
    t.tp_free = PyObject_GC_Del;
    t.tp_dictoffset = offsetof(Entry, dict);
    t.tp_weaklistoffset = offsetof(Entry, weak_references);
    t.tp_descr_get = entry_get;
    t.tp_methods = entry_methods;
    t.tp_getset = entry_attributes;
    return t;
}();

// The C signature decides an argument's kind and how it is passed.
template <class F> struct Signature;
template <class... A> struct Signature<int(A...)> {
    static constexpr int COUNT = sizeof...(A);
    template <class T> static T pass(unsigned long long v) {
        if constexpr (std::is_pointer_v<T>) return reinterpret_cast<T>(static_cast<uintptr_t>(v));
        else return static_cast<T>(v);
    }
    template <size_t... I> static int call(void *f, const unsigned long long *v, std::index_sequence<I...>) {
        return reinterpret_cast<int (*)(A...)>(f)(pass<A>(v[I])...);
    }
    static int invoke(void *f, const unsigned long long *v) { return call(f, v, std::index_sequence_for<A...>{}); }
    static void kinds(Kind *kind) {
        constexpr bool pointer[] = {std::is_pointer_v<A>...};
        for (int i = 0; i < COUNT; i++) kind[i] = pointer[i] ? POINTER : INTEGER;
    }
};

// `names`: the arguments in order; those from position `required` on may be left out (None). The last one
// is the stream.
template <class F>
bool add_entry(PyObject *module, const char *name, int required, std::initializer_list<const char *> names) {
    using S = Signature<F>;
    static_assert(S::COUNT <= MAX_ARGS, "room for the arguments");
    Entry *e = PyObject_GC_New(Entry, &EntryType);
    if (!e) return false;
    e->call = entry_call;
    e->name = name;
    e->function = nullptr;
    e->invoke = S::invoke;
    e->count = 0;
    e->required = required;
    e->dict = e->weak_references = nullptr;
    S::kinds(e->kind);
    e->kind[S::COUNT - 1] = STREAM;
    for (const char *n : names) e->keyword[e->count++] = PyUnicode_InternFromString(n);
    PyObject_GC_Track(reinterpret_cast<PyObject *>(e));
    if (e->count != S::COUNT) {
        PyErr_Format(PyExc_SystemError, "%s: %d names for %d arguments", name, e->count, S::COUNT);
        return false;
    }
    return PyModule_AddObject(module, name, reinterpret_cast<PyObject *>(e)) == 0;
}

// hooks(address, stream, failed, load, current_device, raw_stream)
PyObject *hooks(PyObject *, PyObject *args) {
    PyObject *h[6];
    if (!PyArg_ParseTuple(args, "OOOOOO", &h[0], &h[1], &h[2], &h[3], &h[4], &h[5])) return nullptr;
    PyObject **to[6] = {&g_address, &g_stream, &g_failed, &g_load, &g_current_device, &g_raw_stream};
    for (int i = 0; i < 6; i++) {
        PyObject *value = h[i] == Py_None ? nullptr : h[i];
        Py_XINCREF(value);
        Py_XSETREF(*to[i], value);
    }
    Py_RETURN_NONE;
}

// connect(entry, address)
PyObject *connect(PyObject *, PyObject *args) {
    PyObject *o, *address;
    unsigned long long value;
    if (!PyArg_ParseTuple(args, "O!O", &EntryType, &o, &address) || !as_integer(address, value)) return nullptr;
    reinterpret_cast<Entry *>(o)->function = reinterpret_cast<void *>(static_cast<uintptr_t>(value));
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"hooks", hooks, METH_VARARGS, nullptr}, {"connect", connect, METH_VARARGS, nullptr}, {}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_call", nullptr, -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__call(void) {
    if (PyType_Ready(&EntryType) < 0) return nullptr;
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    PyObject *m = PyModule_Create(&module_def);
    if (!m || !s_data_ptr) return nullptr;
#define ENTRY(NAME, REQUIRED, ...) add_entry<decltype(NAME)>(m, #NAME, REQUIRED, {__VA_ARGS__})
    const bool ok =
        ENTRY(qtip_rht, 7, "x", "signs", "n", "block", "batch", "side", "out", "stream") &&
        ENTRY(qtip_rht_f32, 7, "x", "signs", "n", "block", "batch", "side", "out", "stream") &&
        ENTRY(qtip_decode_matvec, 10, "codes", "L", "k", "V", "code_id", "lut", "m", "n", "x", "y", "stream") &&
        ENTRY(qtip_rht_decode_matvec, 13, "codes", "L", "k", "V", "code_id", "lut", "m", "n", "x", "signs_n", "block",
              "row_scale", "y", "xt_scratch", "stream") &&
        ENTRY(qtip_rht_decode_matvec_noalloc, 13, "codes", "L", "k", "V", "code_id", "lut", "m", "n", "x", "signs_n",
              "block", "row_scale", "y", "stream") &&
        ENTRY(qtip_decode_matmat, 12, "codes", "L", "k", "V", "code_id", "lut", "m", "n", "X", "B", "row_scale", "Y",
              "stream") &&
        ENTRY(qtip_dequantize, 9, "codes", "L", "k", "V", "code_id", "lut", "m", "n", "W", "stream") &&
        ENTRY(qtip_decode_states, 7, "states", "count", "L", "V", "code_id", "lut", "out", "stream") &&
        ENTRY(qtip_quantize_gpu, 12, "W", "m", "n", "L", "k", "V", "code_id", "lut", "codes_out", "tile_err",
              "workspace", "workspace_bytes", "stream") &&
        ENTRY(qtip_block_ldl, 7, "H", "n", "g", "A_out", "D_out", "workspace", "workspace_bytes", "stream") &&
        ENTRY(qtip_quantize_ldlq, 14, "W", "A", "m", "n", "L", "k", "V", "code_id", "lut", "codes_out", "What_out",
              "tile_err", "workspace", "workspace_bytes", "stream");
#undef ENTRY
    return ok ? m : nullptr;
}
