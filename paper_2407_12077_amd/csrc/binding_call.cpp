// The calls of the Python binding in native code (CPython extension `_call`): arguments to C types, the current stream,
// the call, the status.  Where a kernel takes three microseconds the host is what a call costs.  Measured, a decode step of
// one user (32 heads): 5.2 us a call through ctypes, 4.2 here; of the host's part before the library's own checks and
// launch 2.3 us became 0.85, and 0.5 of these are torch's seven data_ptr().  (A first call on new buffers takes 18 to 21 us
// either way.)
// The functions are those of the library that the binding has loaded, found in it by name; their types come from the header,
// so a list of arguments that does not match does not compile.
//
// Conversions are those of ctypes: whole numbers only (whatever has __index__, cut to the C type's width), None or an
// object with data_ptr() for an address, and the interpreter lock is not held during the call.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <dlfcn.h>

#include <tuple>
#include <type_traits>
#include <utility>

#include "wkv6.h"

namespace {

PyObject* g_data_ptr = nullptr;        // "data_ptr"
PyObject* g_failed = nullptr;          // raises for a status
PyObject* g_bad_number = nullptr;      // exception class for a number of the wrong type
PyObject* g_slow_stream = nullptr;     // () -> handle of the current stream, whatever state torch is in
PyObject* g_get_stream = nullptr;      // device -> handle, and
PyObject* g_get_device = nullptr;      // () -> device: set once torch has initialised the GPU

bool whole_number(PyObject* o, unsigned long long* out) {
    if (PyLong_CheckExact(o)) {
        *out = PyLong_AsUnsignedLongLongMask(o);
    } else {
        PyObject* n = PyNumber_Index(o);
        if (!n) {
            if (PyErr_ExceptionMatches(PyExc_TypeError))
                PyErr_Format(g_bad_number, "a whole number is needed, not '%s'", Py_TYPE(o)->tp_name);
            return false;
        }
        *out = PyLong_AsUnsignedLongLongMask(n);
        Py_DECREF(n);
    }
    return !(*out == ~0ull && PyErr_Occurred());
}

bool convert(PyObject* o, int* out) {
    unsigned long long v;
    if (!whole_number(o, &v)) return false;
    *out = static_cast<int>(v);
    return true;
}
bool convert(PyObject* o, long long* out) {
    unsigned long long v;
    if (!whole_number(o, &v)) return false;
    *out = static_cast<long long>(v);
    return true;
}
bool convert(PyObject* o, float* out) {
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) {
        if (PyErr_ExceptionMatches(PyExc_TypeError))
            PyErr_Format(g_bad_number, "a number is needed, not '%s'", Py_TYPE(o)->tp_name);
        return false;
    }
    *out = static_cast<float>(v);
    return true;
}
template <typename T>
bool convert(PyObject* o, T** out) {
    *out = nullptr;
    if (o == Py_None) return true;
    PyObject* address = PyObject_CallMethodNoArgs(o, g_data_ptr);
    if (!address) return false;
    unsigned long long v = 0;
    const bool ok = address == Py_None || whole_number(address, &v);
    Py_DECREF(address);
    *out = reinterpret_cast<T*>(v);
    return ok;
}

bool stream_of(PyObject* o, void** out) {
    PyObject* handle;
    if (o != Py_None) {
        handle = PyNumber_Long(o);
    } else if (g_get_stream) {
        PyObject* get = g_get_stream;
        Py_INCREF(get);                // another thread may set the sources while these run
        PyObject* device = PyObject_CallNoArgs(g_get_device);
        handle = device ? PyObject_CallOneArg(get, device) : nullptr;
        Py_XDECREF(device);
        Py_DECREF(get);
    } else {
        handle = PyObject_CallNoArgs(g_slow_stream);
    }
    if (!handle) return false;
    unsigned long long v;
    const bool ok = whole_number(handle, &v);
    Py_DECREF(handle);
    *out = reinterpret_cast<void*>(v);
    return ok;
}

// every entry point: int f(..., void* stream)
template <typename... A, std::size_t... I>
PyObject* invoke(int (*fn)(A...), const char* name, PyObject* const* args, Py_ssize_t n, std::index_sequence<I...>) {
    constexpr std::size_t kLast = sizeof...(A) - 1;
    static_assert(std::is_same_v<std::tuple_element_t<kLast, std::tuple<A...>>, void*>, "the stream");
    if (!fn) {
        PyErr_Format(PyExc_RuntimeError, "%s: no library bound", name);
        return nullptr;
    }
    if (n != static_cast<Py_ssize_t>(sizeof...(A))) {
        PyErr_Format(PyExc_TypeError, "%s takes %zu arguments (%zd given)", name, sizeof...(A), n);
        return nullptr;
    }
    std::tuple<A...> c;
    const bool ok = ([&] {
        if constexpr (I < kLast) return convert(args[I], &std::get<I>(c));
        else return stream_of(args[I], &std::get<I>(c));
    }() && ...);
    if (!ok) return nullptr;
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = fn(std::get<I>(c)...);
    Py_END_ALLOW_THREADS
    if (status != WKV6_OK) {
        PyObject* r = PyObject_CallFunction(g_failed, "i", status);
        Py_XDECREF(r);
        if (!PyErr_Occurred()) PyErr_Format(PyExc_RuntimeError, "%s: status %d", name, status);
        return nullptr;
    }
    Py_RETURN_NONE;
}
template <typename... A>
PyObject* invoke(int (*fn)(A...), const char* name, PyObject* const* args, Py_ssize_t n) {
    return invoke(fn, name, args, n, std::index_sequence_for<A...>{});
}

#define WKV6_CALLS(X)                                                                                                         \
    X(wkv6_prefill_bf16) X(wkv6_prefill_bf16_f32out) X(wkv6_prefill_bf16_strided) X(wkv6_prefill_f32)                         \
    X(wkv6_prefill_bf16_recurrent) X(wkv6_prefill_bf16_split) X(wkv6_prefill_bf16_split_noalloc) X(wkv6_finch_c2_prefill_bf16) \
    X(wkv6_finch_c2_prefill_bf16_f32out) X(wkv6_finch_c2_prefill_bf16_strided) X(wkv6_finch_c2_prefill_bf16_split)            \
    X(wkv6_finch_c2_prefill_bf16_moments) X(wkv6_layernorm_finalize) X(wkv6_layernorm_apply_bf16)                             \
    X(wkv6_decay_lora_input_bf16) X(wkv6_finch_c2_prefill_lora_bf16) X(wkv6_prefill_lora_bf16) X(wkv6_decode_bf16)            \
    X(wkv6_finch_c2_decode_bf16) X(wkv6_append_bf16) X(wkv6_finch_c2_append_bf16) X(wkv6_key_compress_bf16)

#define X(name)                                                                                    \
    decltype(&::name) fn_##name = nullptr;                                                         \
    PyObject* py_##name(PyObject*, PyObject* const* args, Py_ssize_t n) { return invoke(fn_##name, #name, args, n); }
WKV6_CALLS(X)
#undef X

// bind(handle, failed, slow_stream, bad_number): the functions of the library behind a dlopen handle
PyObject* bind(PyObject*, PyObject* args) {
    unsigned long long handle;
    PyObject *failed, *slow, *bad;
    if (!PyArg_ParseTuple(args, "KOOO", &handle, &failed, &slow, &bad)) return nullptr;
    void* lib = reinterpret_cast<void*>(handle);
#define X(name)                                                                    \
    if (!dlsym(lib, #name)) {                                                      \
        PyErr_SetString(PyExc_AttributeError, "undefined symbol: " #name);         \
        return nullptr;                                                            \
    }
    WKV6_CALLS(X)
#undef X
#define X(name) fn_##name = reinterpret_cast<decltype(fn_##name)>(dlsym(lib, #name));
    WKV6_CALLS(X)
#undef X
    Py_INCREF(failed);
    Py_XSETREF(g_failed, failed);
    Py_INCREF(bad);
    Py_XSETREF(g_bad_number, bad);
    Py_INCREF(slow);
    Py_XSETREF(g_slow_stream, slow);
    Py_RETURN_NONE;
}

// stream_source(get_stream, get_device): the raw accessors; None, None: back to the slow path
PyObject* stream_source(PyObject*, PyObject* args) {
    PyObject *get, *device;
    if (!PyArg_ParseTuple(args, "OO", &get, &device)) return nullptr;
    const bool none = get == Py_None || device == Py_None;
    Py_XINCREF(none ? nullptr : get);
    Py_XSETREF(g_get_stream, none ? nullptr : get);
    Py_XINCREF(none ? nullptr : device);
    Py_XSETREF(g_get_device, none ? nullptr : device);
    Py_RETURN_NONE;
}

#define X(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_##name)), METH_FASTCALL, nullptr},
PyMethodDef methods[] = {WKV6_CALLS(X){"bind", bind, METH_VARARGS, nullptr},
                         {"stream_source", stream_source, METH_VARARGS, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
#undef X

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__call(void) {
    g_data_ptr = PyUnicode_InternFromString("data_ptr");
    if (!g_data_ptr) return nullptr;
    return PyModule_Create(&module);
}
