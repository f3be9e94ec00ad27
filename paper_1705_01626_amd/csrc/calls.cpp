// Python entry to the device calls of libzvc (include/zvc.h): the same arguments as
// the C functions, as integers, and the status as the result.  A call through
// ctypes converts its nine or ten arguments one object at a time, 3 us of a call
// whose kernel takes 4; here they are read from the interpreter's argument array.
// The interpreter lock is released during the call, as ctypes does.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include "zvc.h"

#include <dlfcn.h>

#include <cstdint>
#include <type_traits>
#include <utility>

namespace {

// One integer argument as the C type of the parameter (modulo 2^64, as a C caller's conversion would be).
template <typename T>
T from_word(unsigned long long v) {
    if constexpr (std::is_pointer_v<T>) return reinterpret_cast<T>(static_cast<uintptr_t>(v));
    else return static_cast<T>(v);
}

template <typename R, typename... Params, size_t... I>
R call(R (*f)(Params...), const unsigned long long* words, std::index_sequence<I...>) {
    return f(from_word<Params>(words[I])...);
}

// The functions of the library that open() was given, one slot per function.
template <auto F>
decltype(F) g_function = nullptr;

// Raised for an argument that is no integer: ctypes.ArgumentError, as before this module, and a TypeError.
PyObject* g_argument_error = nullptr;

template <auto F, typename R, typename... Params>
PyObject* forward(R (*)(Params...), PyObject* const* args, Py_ssize_t count) {
    constexpr Py_ssize_t kParams = sizeof...(Params);
    if (g_function<F> == nullptr) {
        PyErr_SetString(PyExc_RuntimeError, "open() has not been called");
        return nullptr;
    }
    if (count != kParams) {
        PyErr_Format(PyExc_TypeError, "%zd arguments expected, %zd given", kParams, count);
        return nullptr;
    }
    unsigned long long words[kParams];
    for (Py_ssize_t i = 0; i < kParams; ++i) {
        words[i] = PyLong_AsUnsignedLongLongMask(args[i]);
        if (words[i] == ~0ull && PyErr_Occurred()) {
            if (PyErr_ExceptionMatches(PyExc_TypeError)) {
                PyErr_Clear();
                PyErr_Format(g_argument_error, "argument %zd: an integer expected, %s given", i + 1,
                             Py_TYPE(args[i])->tp_name);
            }
            return nullptr;
        }
    }
    R result;
    Py_BEGIN_ALLOW_THREADS
    result = call(g_function<F>, words, std::index_sequence_for<Params...>{});
    Py_END_ALLOW_THREADS
    return PyLong_FromUnsignedLongLong(static_cast<unsigned long long>(result));
}

template <auto F>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t count) {
    return forward<F>(F, args, count);
}

template <auto F>
bool bind(void* library, const char* name) {
    g_function<F> = reinterpret_cast<decltype(F)>(dlsym(library, name));
    if (g_function<F> == nullptr) PyErr_Format(PyExc_ImportError, "%s is not in the library", name);
    return g_function<F> != nullptr;
}

#define ZVC_FUNCTIONS(DO)                                                                       \
    DO(zvc_compressed_size) DO(zvc_compress) DO(zvc_compress_static) DO(zvc_relu_compress)      \
    DO(zvc_compress_bounded) DO(zvc_decompress) DO(zvc_window_elements) DO(zvc_window_count)    \
    DO(zvc_window_compress) DO(zvc_window_decompress) DO(zvc_offload) DO(zvc_relu_offload)      \
    DO(zvc_prefetch)

// open(path): take the functions from the library at `path` (normally one that is loaded already).
PyObject* open_library(PyObject*, PyObject* path) {
    PyObject* bytes = nullptr;
    if (!PyUnicode_FSConverter(path, &bytes)) return nullptr;
    void* library = dlopen(PyBytes_AS_STRING(bytes), RTLD_NOW | RTLD_LOCAL);
    Py_DECREF(bytes);
    if (library == nullptr) {
        PyErr_SetString(PyExc_ImportError, dlerror());
        return nullptr;
    }
#define ZVC_BIND(NAME) if (!bind<&NAME>(library, #NAME)) return nullptr;
    ZVC_FUNCTIONS(ZVC_BIND)
#undef ZVC_BIND
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"open", open_library, METH_O, nullptr},
#define ZVC_ENTRY(NAME) \
    {#NAME, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&entry<&NAME>)), METH_FASTCALL, nullptr},
    ZVC_FUNCTIONS(ZVC_ENTRY)
#undef ZVC_ENTRY
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls() {
    PyObject* ctypes = PyImport_ImportModule("ctypes");
    if (ctypes == nullptr) return nullptr;
    PyObject* base = PyObject_GetAttrString(ctypes, "ArgumentError");
    Py_DECREF(ctypes);
    if (base == nullptr) return nullptr;
    PyObject* bases = PyTuple_Pack(2, base, PyExc_TypeError);
    Py_DECREF(base);
    if (bases == nullptr) return nullptr;
    g_argument_error = PyErr_NewException("paper_1705_01626_amd._calls.ArgumentError", bases, nullptr);
    Py_DECREF(bases);
    return g_argument_error == nullptr ? nullptr : PyModule_Create(&module);
}
