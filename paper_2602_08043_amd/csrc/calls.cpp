// Python arguments -> calls of the C ABI (include/vabft.h).  A call of the session has 9 to 24 arguments; marshalled by
// ctypes, with data_ptr() of every tensor called from Python, it took 8 to 9 us of host time, more than the GPU needs for a
// small product (f32 256^3, two calls: 16.5 us a pass on the host, 12.8 on the GPU).  Converted here it takes 4 to 5, most of
// it the launch.  Pointers may be tensors (anything with data_ptr()), integers, None or what ctypes takes for a c_void_p;
// structures are the binding's own.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstring>
#include <tuple>
#include <type_traits>
#include <utility>

#include "vabft.h"

namespace {

PyObject* g_data_ptr;  // "data_ptr"
PyObject* g_value;     // "value"
PyObject* g_cast;      // ctypes.cast, ctypes.c_void_p, ctypes.c_size_t
PyObject* g_void_p;
PyObject* g_size_t;
PyObject* g_problem;   // the binding's structures
PyObject* g_inject;

bool to_address(PyObject* o, void** out) {
    if (o == Py_None) {
        *out = nullptr;
        return true;
    }
    if (PyLong_Check(o)) {
        *out = PyLong_AsVoidPtr(o);
        return !PyErr_Occurred();
    }
    PyObject* r = PyObject_CallMethodNoArgs(o, g_data_ptr);
    if (!r && PyErr_ExceptionMatches(PyExc_AttributeError) && !PyUnicode_Check(o) && !PyBytes_Check(o)) {
        // what ctypes takes for a c_void_p: pointers, arrays, byref(); of anything else it makes an ArgumentError
        PyErr_Clear();
        PyObject* const p = PyObject_CallFunctionObjArgs(g_cast, o, g_void_p, nullptr);
        r = p ? PyObject_GetAttr(p, g_value) : nullptr;
        Py_XDECREF(p);
    }
    if (!r) return false;
    const bool ok = r == Py_None || PyLong_Check(r);
    *out = ok && r != Py_None ? PyLong_AsVoidPtr(r) : nullptr;
    Py_DECREF(r);
    if (!ok) PyErr_SetString(PyExc_TypeError, "data_ptr() must give an integer");
    return ok && !PyErr_Occurred();
}

// the memory of one of the binding's structures, which its owner keeps for the length of the call
bool to_struct(PyObject* o, PyObject* type, size_t bytes, const void** out) {
    *out = nullptr;
    if (o == Py_None) return true;
    const int is = type ? PyObject_IsInstance(o, type) : 0;
    if (is < 0) return false;
    Py_buffer view;
    if (!is || PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_TypeError, "a structure of another type");
        return false;
    }
    const bool ok = (size_t)view.len >= bytes;
    *out = view.buf;
    PyBuffer_Release(&view);
    if (!ok) PyErr_SetString(PyExc_TypeError, "structure of another size");
    return ok;
}

// float(o)
bool to_double(PyObject* o, double* out) {
    PyObject* const f = PyFloat_CheckExact(o) ? nullptr : PyNumber_Float(o);
    if (!f && PyErr_Occurred()) return false;
    *out = PyFloat_AS_DOUBLE(f ? f : o);
    Py_XDECREF(f);
    return true;
}

// an integer, or a ctypes.c_size_t
bool to_size(PyObject* o, size_t* out) {
    PyObject* r = nullptr;
    if (!PyLong_Check(o)) {
        const int is = PyObject_IsInstance(o, g_size_t);
        if (is < 0 || (is && !(r = PyObject_GetAttr(o, g_value)))) return false;
    }
    *out = PyLong_AsSize_t(r ? r : o);
    Py_XDECREF(r);
    return !(*out == (size_t)-1 && PyErr_Occurred());
}

template <typename T> bool convert(PyObject* o, T* out) {
    if constexpr (std::is_same<T, const vabft_problem*>::value || std::is_same<T, const vabft_inject*>::value) {
        const void* p;
        if (!to_struct(o, std::is_same<T, const vabft_problem*>::value ? g_problem : g_inject, sizeof(**out), &p)) return false;
        *out = static_cast<T>(p);
    } else if constexpr (std::is_pointer<T>::value) {
        void* p;
        if (!to_address(o, &p)) return false;
        *out = static_cast<T>(p);
    } else if constexpr (std::is_floating_point<T>::value) {
        return to_double(o, out);
    } else if constexpr (std::is_same<T, size_t>::value) {
        return to_size(o, out);
    } else {
        static_assert(std::is_same<T, int32_t>::value, "a type of the ABI");
        const long v = PyLong_AsLong(o);
        if (v == -1 && PyErr_Occurred()) return false;
        if (v != (long)(int32_t)v) {
            PyErr_SetString(PyExc_OverflowError, "does not fit 32 bits");
            return false;
        }
        *out = (int32_t)v;
    }
    return true;
}

template <typename... A, size_t... I>
PyObject* call(int (*f)(A...), const char* name, PyObject* const* args, Py_ssize_t n, std::index_sequence<I...>) {
    if (n != (Py_ssize_t)sizeof...(A)) {
        PyErr_Format(PyExc_TypeError, "%s takes %d arguments, not %d", name, (int)sizeof...(A), (int)n);
        return nullptr;
    }
    std::tuple<A...> v{};
    if (!(convert(args[I], &std::get<I>(v)) && ...)) return nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS;
    rc = f(std::get<I>(v)...);
    Py_END_ALLOW_THREADS;
    return PyLong_FromLong(rc);
}
template <typename... A> PyObject* call(int (*f)(A...), const char* name, PyObject* const* args, Py_ssize_t n) {
    return call(f, name, args, n, std::index_sequence_for<A...>{});
}

// one method per entry point; its self is the entry point's address in the library that was loaded
#define ENTRY(NAME)                                                                            \
    PyObject* py_##NAME(PyObject* self, PyObject* const* args, Py_ssize_t n) {                 \
        return call(reinterpret_cast<decltype(&NAME)>(PyLong_AsVoidPtr(self)), #NAME, args, n); \
    }
#define ENTRIES(X)                                                                                                     \
    X(vabft_workspace_init) X(vabft_encode) X(vabft_threshold) X(vabft_gemm_verified) X(vabft_gemm_verified_fused)     \
    X(vabft_gemm_verified_fused_static) X(vabft_encode_weighted) X(vabft_threshold_weighted)                           \
    X(vabft_gemm_verified_weighted) X(vabft_locate_correct) X(vabft_check_offline) X(vabft_encode_a)                   \
    X(vabft_threshold_cols) X(vabft_gemm_verified_rc) X(vabft_encode_blocks) X(vabft_threshold_blocks)                 \
    X(vabft_gemm_verified_blocks) X(vabft_encode_blocks_k) X(vabft_threshold_blocks_k) X(vabft_gemm_verified_blocks_k) \
    X(vabft_encode_gemm_fused) X(vabft_encode_gemm_weighted)
ENTRIES(ENTRY)

#define METHOD(NAME) {#NAME, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(py_##NAME)), METH_FASTCALL, nullptr},
PyMethodDef g_entries[] = {ENTRIES(METHOD){nullptr, nullptr, 0, nullptr}};

PyObject* bind(PyObject*, PyObject* args) {
    const char* name;
    PyObject* address;
    if (!PyArg_ParseTuple(args, "sO!", &name, &PyLong_Type, &address)) return nullptr;
    for (PyMethodDef* m = g_entries; m->ml_name; ++m)
        if (!strcmp(m->ml_name, name)) return PyCFunction_New(m, address);
    return PyErr_Format(PyExc_KeyError, "no entry point %s", name);
}

PyObject* structures(PyObject*, PyObject* args) {
    PyObject *problem, *inject;
    if (!PyArg_ParseTuple(args, "O!O!", &PyType_Type, &problem, &PyType_Type, &inject)) return nullptr;
    Py_INCREF(problem);
    Py_INCREF(inject);
    Py_XSETREF(g_problem, problem);
    Py_XSETREF(g_inject, inject);
    Py_RETURN_NONE;
}

PyMethodDef g_methods[] = {
    {"structures", structures, METH_VARARGS, "structures(Problem, Inject): the ctypes classes of vabft_problem and vabft_inject"},
    {"bind", bind, METH_VARARGS, "bind(name, address): the entry point at an address as a Python callable"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_calls", "Native calls of libvabft's entry points.", -1, g_methods,
                        nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls(void) {
    g_data_ptr = PyUnicode_InternFromString("data_ptr");
    g_value = PyUnicode_InternFromString("value");
    PyObject* const ctypes = PyImport_ImportModule("ctypes");
    g_cast = ctypes ? PyObject_GetAttrString(ctypes, "cast") : nullptr;
    g_void_p = ctypes ? PyObject_GetAttrString(ctypes, "c_void_p") : nullptr;
    g_size_t = ctypes ? PyObject_GetAttrString(ctypes, "c_size_t") : nullptr;
    Py_XDECREF(ctypes);
    PyObject* m = g_data_ptr && g_value && g_cast && g_void_p && g_size_t ? PyModule_Create(&g_module) : nullptr;
    PyObject* names = m ? PyList_New(0) : nullptr;
    for (PyMethodDef* e = g_entries; names && e->ml_name; ++e) {
        PyObject* s = PyUnicode_FromString(e->ml_name);
        if (!s || PyList_Append(names, s) != 0) Py_CLEAR(names);
        Py_XDECREF(s);
    }
    if (!names || PyModule_AddObject(m, "ENTRIES", names) != 0) return nullptr;
    return m;
}
