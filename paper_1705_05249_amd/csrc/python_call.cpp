// The calls of gemm.py without ctypes: one C function per entry point that takes the Python arguments as they are (tensors, addresses,
// None), asks tensors for their addresses and torch for its current stream, and calls the library with the interpreter's lock released.
// In ctypes and Python these conversions were 4 us of the 7.6 that the host took for a small product, 0.9 of 3.8 now: calls one behind the other,
// FP32 256^3 7.6 -> 4.8 us, which is the kernel's own time, FP16 64 x 64 x 64 7.6 -> 3.8.
//
// Arguments of other types (ctypes' own scalars, objects that only ctypes can convert, errors) go to gemm.py, which makes the call through ctypes.
//
// The library is not linked: gemm.py loads it and hands over the addresses of its functions (bind).  Conversions follow from the entry points'
// own types: a size_t stands for the bytes of the workspace in front of it, the last pointer is the stream.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <stddef.h>
#include <stdint.h>

#include <tuple>
#include <type_traits>
#include <utility>

#include "../../include/mg_gemm.h"

namespace {

PyObject *s_data_ptr, *s_numel, *s_element_size, *s_cuda_stream;       // interned names
PyObject *stream_calls;                     // gemm.py's: () -> torch's functions for the current device and for its current stream
PyObject *get_device, *get_stream;          // these
PyObject *other_types;                      // gemm.py's: (name, arguments) -> status, through ctypes

// an address: None, an integer, or a tensor
bool address(PyObject *o, void **out)
{
    if (o == Py_None) {
        *out = nullptr;
        return true;
    }
    PyObject *held = nullptr;
    if (!PyLong_Check(o)) {
        held = PyObject_CallMethodNoArgs(o, s_data_ptr);
        if (held == nullptr) return false;
        o = held;
    }
    const unsigned long long v = PyLong_AsUnsignedLongLongMask(o);
    Py_XDECREF(held);
    if (v == static_cast<unsigned long long>(-1) && PyErr_Occurred()) return false;
    *out = reinterpret_cast<void *>(static_cast<uintptr_t>(v));
    return true;
}

// the address of torch's current stream on its current device
PyObject *current_stream()
{
    if (get_stream == nullptr) {
        PyObject *calls = PyObject_CallNoArgs(stream_calls);
        if (calls == nullptr) return nullptr;
        if (!PyArg_ParseTuple(calls, "OO", &get_device, &get_stream)) {
            Py_DECREF(calls);
            return nullptr;
        }
        Py_INCREF(get_device);          // (kept until the process ends, as the module is)
        Py_INCREF(get_stream);
        Py_DECREF(calls);
    }
    PyObject *device = PyObject_CallNoArgs(get_device);
    if (device == nullptr) return nullptr;
    PyObject *stream = PyObject_CallOneArg(get_stream, device);
    Py_DECREF(device);
    return stream;
}

// None (torch's current stream), an integer, or an object with an attribute cuda_stream
bool stream_address(PyObject *o, void **out)
{
    PyObject *held = nullptr;
    if (o == Py_None) held = current_stream();
    else if (PyLong_Check(o)) return address(o, out);
    else if (PyObject_HasAttr(o, s_cuda_stream)) held = PyObject_GetAttr(o, s_cuda_stream);
    else return address(o, out);
    if (held == nullptr) return false;
    const bool ok = address(held, out);
    Py_DECREF(held);
    return ok;
}

// numel() * element_size() of a workspace tensor
bool workspace_bytes(PyObject *o, size_t *out)
{
    *out = 0;
    if (o == Py_None) return true;
    size_t product = 1;
    for (PyObject *name : {s_numel, s_element_size}) {
        PyObject *v = PyObject_CallMethodNoArgs(o, name);
        if (v == nullptr) return false;
        product *= PyLong_AsSize_t(v);
        Py_DECREF(v);
        if (PyErr_Occurred() != nullptr) return false;
    }
    *out = product;
    return true;
}

template <typename P> bool convert(PyObject *o, bool last, P *out)
{
    if constexpr (std::is_pointer_v<P>) {
        void *v = nullptr;
        if (!(last ? stream_address(o, &v) : address(o, &v))) return false;
        *out = static_cast<P>(v);
        return true;
    } else if constexpr (std::is_same_v<P, size_t>) {
        return workspace_bytes(o, out);
    } else if constexpr (std::is_floating_point_v<P>) {
        const double v = PyFloat_AsDouble(o);
        *out = static_cast<P>(v);
        return v != -1.0 || PyErr_Occurred() == nullptr;
    } else {
        if (!PyLong_Check(o)) {
            PyErr_Format(PyExc_TypeError, "int expected instead of %.100s instance", Py_TYPE(o)->tp_name);
            return false;
        }
        *out = static_cast<P>(PyLong_AsUnsignedLongLongMask(o));
        return true;
    }
}

// Python arguments in front of parameter i: all but the size_t, which shares the workspace's
template <typename... P> constexpr Py_ssize_t arguments_before(size_t i)
{
    constexpr bool counted[] = {!std::is_same_v<P, size_t>...};
    Py_ssize_t n = 0;
    for (size_t j = 0; j < i; ++j) n += counted[j];
    return n;
}

// what is left of a call that cannot be converted here: the error, or what ctypes makes of it
PyObject *call_other_types(const char *name, PyObject *const *args, Py_ssize_t count)
{
    if (other_types == nullptr || !(PyErr_ExceptionMatches(PyExc_TypeError) || PyErr_ExceptionMatches(PyExc_OverflowError))) return nullptr;
    PyErr_Clear();
    PyObject *list = PyTuple_New(count);
    if (list == nullptr) return nullptr;
    for (Py_ssize_t i = 0; i < count; ++i) {
        Py_INCREF(args[i]);
        PyTuple_SET_ITEM(list, i, args[i]);
    }
    PyObject *status = PyObject_CallFunction(other_types, "sN", name, list);
    return status;
}

template <typename... P, size_t... I>
PyObject *invoke(const char *name, mg_status (*fn)(P...), PyObject *const *args, Py_ssize_t count, std::index_sequence<I...>)
{
    constexpr Py_ssize_t wanted = arguments_before<P...>(sizeof...(P));
    if (count != wanted || fn == nullptr) {
        PyErr_Format(PyExc_TypeError, fn == nullptr ? "the library is not bound" : "%zd arguments expected, not %zd", wanted, count);
        return nullptr;
    }
    std::tuple<P...> v;
    if (!(convert<P>(args[std::is_same_v<P, size_t> ? arguments_before<P...>(I) - 1 : arguments_before<P...>(I)], I + 1 == sizeof...(P), &std::get<I>(v)) && ...))
        return call_other_types(name, args, count);
    mg_status status;
    Py_BEGIN_ALLOW_THREADS
    status = fn(std::get<I>(v)...);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(static_cast<long>(status));
}

#define MG_ENTRIES(X)                                                                                                       \
    X(mg_sgemm) X(mg_hgemm) X(mg_sgemm_static) X(mg_sgemv) X(mg_hgemv) X(mg_ssymm) X(mg_hsymm) X(mg_ssyrk) X(mg_hsyrk)      \
    X(mg_strmm) X(mg_htrmm) X(mg_sgemm_batched) X(mg_hgemm_batched) X(mg_sgemm_strided_batched) X(mg_hgemm_strided_batched) \
    X(mg_sim2col) X(mg_him2col) X(mg_sconv2d) X(mg_hconv2d)

#define X(name)                                                                                 \
    decltype(&::name) bound_##name;                                                             \
    template <typename... P> PyObject *call_##name(mg_status (*fn)(P...), PyObject *const *args, Py_ssize_t count) \
    {                                                                                           \
        return invoke(#name, fn, args, count, std::index_sequence_for<P...>{});                 \
    }                                                                                           \
    PyObject *py_##name(PyObject *, PyObject *const *args, Py_ssize_t count) { return call_##name(bound_##name, args, count); }
MG_ENTRIES(X)
#undef X

// bind(name -> address, stream_calls[, other_types])
PyObject *bind(PyObject *, PyObject *const *args, Py_ssize_t count)
{
    if ((count != 2 && count != 3) || !PyDict_Check(args[0])) {
        PyErr_SetString(PyExc_TypeError, "bind(addresses, stream_calls[, other_types])");
        return nullptr;
    }
    void *at = nullptr;
#define X(name)                                                                       \
    if (PyObject *o = PyDict_GetItemString(args[0], #name)) {                          \
        if (!address(o, &at)) return nullptr;                                          \
        bound_##name = reinterpret_cast<decltype(&::name)>(at);                        \
    }
    MG_ENTRIES(X)
#undef X
    Py_INCREF(args[1]);
    Py_XSETREF(stream_calls, args[1]);
    if (count == 3) {
        Py_INCREF(args[2]);
        Py_XSETREF(other_types, args[2]);
    }
    Py_RETURN_NONE;
}

#define X(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_##name)), METH_FASTCALL, nullptr},
PyMethodDef methods[] = {MG_ENTRIES(X){"bind", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(bind)), METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
#undef X

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_mg_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__mg_call()
{
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_numel = PyUnicode_InternFromString("numel");
    s_element_size = PyUnicode_InternFromString("element_size");
    s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    if (s_data_ptr == nullptr || s_numel == nullptr || s_element_size == nullptr || s_cuda_stream == nullptr) return nullptr;
    return PyModule_Create(&module);
}
