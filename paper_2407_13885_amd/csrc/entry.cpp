// The entry points of libattnw.so as Python callables: arguments as programs pass them (tensors or addresses, whole numbers, a stream) go
// straight to the C function, everything else (other number types, a library not loaded yet) to the Python function that the
// callable stands for.  Behind a public function of the same signature (binding.py): copying, pickling, inspecting and binding are a function's.
//
// What bounds a small call is the host: 7.7 us for one fp32 head of 128 tokens, of which 2.8 are torch.cuda.current_stream(), 3.5 the launch
// and 1.3 the marshalling through ctypes; here 0.3, the function in front 0.07.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <structmember.h>

#include <climits>
#include <cstddef>
#include <cstdint>

namespace {

typedef int64_t i64;

struct Entry {
    PyObject_HEAD
    vectorcallfunc call;
    PyObject* any;        // the Python function
    PyObject* check;      // raises for a status that is not 0
    void* fn;             // the C function, once the library is loaded
    int pointers, sizes, has_scale, dtypes;
};

PyObject *s_data_ptr, *s_cuda_stream;

// 1: converted, 0: not of the expected kind, -1: an exception is set
int address(PyObject* x, PyObject* attribute, bool method, void** out)
{
    if (x == Py_None) {
        *out = nullptr;
        return 1;
    }
    if (PyLong_CheckExact(x)) {
        *out = reinterpret_cast<void*>(static_cast<uintptr_t>(PyLong_AsUnsignedLongLongMask(x)));
        return PyErr_Occurred() ? -1 : 1;
    }
    PyObject* v = method ? PyObject_CallMethodNoArgs(x, attribute) : PyObject_GetAttr(x, attribute);
    if (!v) {
        if (!PyErr_ExceptionMatches(PyExc_AttributeError)) return -1;
        PyErr_Clear();
        return 0;
    }
    const int kind = PyLong_CheckExact(v) ? 1 : 0;
    if (kind) *out = reinterpret_cast<void*>(static_cast<uintptr_t>(PyLong_AsUnsignedLongLongMask(v)));
    Py_DECREF(v);
    return PyErr_Occurred() ? -1 : kind;
}

int whole(PyObject* x, i64* out)
{
    if (!PyLong_CheckExact(x)) return 0;
    int overflow = 0;
    *out = PyLong_AsLongLongAndOverflow(x, &overflow);
    return overflow ? 0 : 1;
}

int invoke(const Entry* e, void* const* p, const i64* n, float scale, const int* t, void* stream)
{
    if (e->pointers == 4)
        return reinterpret_cast<int (*)(void*, void*, void*, void*, i64, i64, i64, i64, float, int, void*)>(e->fn)(p[0], p[1], p[2], p[3], n[0],
                                                                                                            n[1], n[2], n[3], scale, t[0], stream);
    if (e->pointers == 3)
        return reinterpret_cast<int (*)(void*, void*, void*, i64, i64, i64, i64, float, int, void*)>(e->fn)(p[0], p[1], p[2], n[0], n[1], n[2],
                                                                                                     n[3], scale, t[0], stream);
    if (e->has_scale) return reinterpret_cast<int (*)(void*, void*, i64, float, int, void*)>(e->fn)(p[0], p[1], n[0], scale, t[0], stream);
    if (e->dtypes == 2) return reinterpret_cast<int (*)(void*, void*, i64, i64, int, int, void*)>(e->fn)(p[0], p[1], n[0], n[1], t[0], t[1], stream);
    return reinterpret_cast<int (*)(void*, void*, i64, i64, int, void*)>(e->fn)(p[0], p[1], n[0], n[1], t[0], stream);
}

PyObject* entry_call(PyObject* self, PyObject* const* args, size_t nargsf, PyObject* names)
{
    Entry* const e = reinterpret_cast<Entry*>(self);
    const Py_ssize_t given = PyVectorcall_NARGS(nargsf);
    const Py_ssize_t required = e->pointers + e->sizes + e->has_scale + e->dtypes;
    if (e->fn && (!names || PyTuple_GET_SIZE(names) == 0) && (given == required || given == required + 1)) {
        void *p[4], *stream = nullptr;
        i64 n[4];
        int t[2], ok = 1;
        float scale = 0.0f;
        PyObject* const* a = args;
        for (int i = 0; ok > 0 && i < e->pointers; ++i) ok = address(*a++, s_data_ptr, true, &p[i]);
        for (int i = 0; ok > 0 && i < e->sizes; ++i) ok = whole(*a++, &n[i]);
        if (ok > 0 && e->has_scale) {
            PyObject* const x = *a++;
            ok = PyFloat_CheckExact(x) ? 1 : 0;
            if (ok) scale = static_cast<float>(PyFloat_AS_DOUBLE(x));
        }
        for (int i = 0; ok > 0 && i < e->dtypes; ++i) {
            i64 v = 0;
            ok = whole(*a++, &v);
            if (ok > 0 && (v < INT_MIN || v > INT_MAX)) ok = 0;
            t[i] = static_cast<int>(v);
        }
        if (ok > 0 && given > required) ok = address(*a, s_cuda_stream, false, &stream);
        if (ok < 0) return nullptr;
        if (ok > 0) {
            int status;
            Py_BEGIN_ALLOW_THREADS
            status = invoke(e, p, n, scale, t, stream);
            Py_END_ALLOW_THREADS
            if (status == 0) Py_RETURN_NONE;
            PyObject* const code = PyLong_FromLong(status);
            if (!code) return nullptr;
            PyObject* const r = PyObject_CallOneArg(e->check, code);
            Py_DECREF(code);
            return r;
        }
    }
    return PyObject_Vectorcall(e->any, args, nargsf, names);
}

// Entry(function, check, pointers, sizes, has_scale, dtypes)
int entry_init(PyObject* self, PyObject* args, PyObject*)
{
    Entry* const e = reinterpret_cast<Entry*>(self);
    PyObject *any, *check;
    if (!PyArg_ParseTuple(args, "OOiiii", &any, &check, &e->pointers, &e->sizes, &e->has_scale, &e->dtypes)) return -1;
    if (e->pointers < 2 || e->pointers > 4 || e->sizes < 1 || e->sizes > 4 || e->dtypes < 1 || e->dtypes > 2) {
        PyErr_SetString(PyExc_ValueError, "no such entry point");
        return -1;
    }
    Py_XSETREF(e->any, Py_NewRef(any));
    Py_XSETREF(e->check, Py_NewRef(check));
    e->fn = nullptr;
    e->call = entry_call;
    return 0;
}

PyObject* entry_bind(PyObject* self, PyObject* arg)
{
    void* const fn = PyLong_AsVoidPtr(arg);
    if (PyErr_Occurred()) return nullptr;
    reinterpret_cast<Entry*>(self)->fn = fn;
    Py_RETURN_NONE;
}

int entry_traverse(PyObject* self, visitproc visit, void* arg)
{
    Entry* const e = reinterpret_cast<Entry*>(self);
    Py_VISIT(e->any);
    Py_VISIT(e->check);
    return 0;
}

int entry_clear(PyObject* self)
{
    Entry* const e = reinterpret_cast<Entry*>(self);
    Py_CLEAR(e->any);
    Py_CLEAR(e->check);
    return 0;
}

void entry_dealloc(PyObject* self)
{
    PyObject_GC_UnTrack(self);
    entry_clear(self);
    Py_TYPE(self)->tp_free(self);
}

PyMethodDef entry_methods[] = {{"bind", entry_bind, METH_O, "bind(address): the C function, from now on called directly"},
                               {nullptr, nullptr, 0, nullptr}};

PyTypeObject entry_type = {PyVarObject_HEAD_INIT(nullptr, 0)};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_entry", "Entry points of libattnw.so as Python callables.", -1, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__entry(void)
{
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    if (!s_data_ptr || !s_cuda_stream) return nullptr;
    entry_type.tp_name = "paper_2407_13885_amd._entry.Entry";
    entry_type.tp_basicsize = sizeof(Entry);
    entry_type.tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_VECTORCALL | Py_TPFLAGS_HAVE_GC;
    entry_type.tp_vectorcall_offset = offsetof(Entry, call);
    entry_type.tp_call = PyVectorcall_Call;
    entry_type.tp_new = PyType_GenericNew;
    entry_type.tp_init = entry_init;
    entry_type.tp_dealloc = entry_dealloc;
    entry_type.tp_traverse = entry_traverse;
    entry_type.tp_clear = entry_clear;
    entry_type.tp_methods = entry_methods;
    if (PyType_Ready(&entry_type) < 0) return nullptr;
    PyObject* const m = PyModule_Create(&module_def);
    if (!m) return nullptr;
    if (PyModule_AddObject(m, "Entry", Py_NewRef(reinterpret_cast<PyObject*>(&entry_type))) < 0) return nullptr;
    return m;
}
