// CPython extension `_native`: the operator entry points of tir.h as builtin functions with positional arguments.
//
// A launch of a microsecond kernel is bound by what the host does per call.  Marshalling seventeen arguments through
// ctypes and asking torch.cuda.current_stream() for its handle took 5.4 us of the 7.5 us of a 128-cube GEMM call; here a
// tensor costs one data_ptr() call, a number one integer conversion and the current stream one torch._C function
// (3.0 us for the same call, 2.3 of them the HIP launch).
//
// Conversions by C parameter type: pointers take a tensor (its data_ptr()), an integer address or None; tir_dtype a
// code or a name ("f16", ...); const tir_epilogue* None or an instance of the binding's Epilogue (set_epilogue_type); the last argument, the
// stream, None (torch's current stream), an integer handle or an object with .cuda_stream.  Every function returns the
// tir_status as an int; wrong argument types raise.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <limits>
#include <tuple>
#include <type_traits>
#include <utility>

#include "tir.h"

namespace {

PyObject* g_data_ptr = nullptr;       // interned method / attribute names
PyObject* g_cuda_stream = nullptr;
PyObject* g_current_stream = nullptr; // torch.cuda.current_stream: initialises the device, used for the first None
PyObject* g_get_device = nullptr;     // torch._C._cuda_getDevice, torch._C._cuda_getCurrentRawStream
PyObject* g_raw_stream = nullptr;
PyObject* g_epilogue_type = nullptr;  // the ctypes structure that mirrors tir_epilogue
bool g_cuda_ready = false;

bool to_address(PyObject* o, void** out) {
    if (o == Py_None) {
        *out = nullptr;
        return true;
    }
    if (PyLong_Check(o)) {
        *out = PyLong_AsVoidPtr(o);
        return !(*out == nullptr && PyErr_Occurred());
    }
    PyObject* r = PyObject_CallMethodNoArgs(o, g_data_ptr);
    if (!r) return false;
    *out = PyLong_AsVoidPtr(r);
    Py_DECREF(r);
    return !(*out == nullptr && PyErr_Occurred());
}

bool to_stream(PyObject* o, void** out) {
    if (o == Py_None) {
        if (!g_cuda_ready) {
            PyObject* s = PyObject_CallNoArgs(g_current_stream);
            if (!s) return false;
            Py_DECREF(s);
            g_cuda_ready = true;
        }
        PyObject* dev = PyObject_CallNoArgs(g_get_device);
        if (!dev) return false;
        PyObject* r = PyObject_CallOneArg(g_raw_stream, dev);
        Py_DECREF(dev);
        if (!r) return false;
        *out = PyLong_AsVoidPtr(r);
        Py_DECREF(r);
        return !(*out == nullptr && PyErr_Occurred());
    }
    if (PyLong_Check(o)) return to_address(o, out);
    PyObject* r = PyObject_GetAttr(o, g_cuda_stream);
    if (!r) return false;
    *out = PyLong_AsVoidPtr(r);
    Py_DECREF(r);
    return !(*out == nullptr && PyErr_Occurred());
}

// One converter per C parameter type; `view` keeps an epilogue's buffer until the call has returned.
struct Held {
    Py_buffer view;
    bool used = false;
    ~Held() {
        if (used) PyBuffer_Release(&view);
    }
};
bool convert(PyObject* o, const void** out, Held&) { return to_address(o, const_cast<void**>(out)); }
bool convert(PyObject* o, void** out, Held&) { return to_address(o, out); }
bool convert(PyObject* o, int64_t* out, Held&) {
    *out = PyLong_AsLongLong(o);
    return !(*out == -1 && PyErr_Occurred());
}
bool convert(PyObject* o, int* out, Held&) {
    const long v = PyLong_AsLong(o);
    if (v == -1 && PyErr_Occurred()) return false;
    if (v < std::numeric_limits<int>::min() || v > std::numeric_limits<int>::max()) {
        PyErr_SetString(PyExc_OverflowError, "argument does not fit a C int");
        return false;
    }
    *out = (int)v;
    return true;
}
bool convert(PyObject* o, float* out, Held&) {
    const double v = PyFloat_AsDouble(o);
    *out = (float)v;
    return !(v == -1.0 && PyErr_Occurred());
}
bool convert(PyObject* o, tir_dtype* out, Held& h) {
    if (PyUnicode_Check(o)) {
        static const struct { const char* name; tir_dtype code; } kNames[] = {
            {"f16", TIR_F16}, {"bf16", TIR_BF16}, {"i8", TIR_I8}, {"f32", TIR_F32}, {"i32", TIR_I32}};
        for (const auto& k : kNames)
            if (PyUnicode_CompareWithASCIIString(o, k.name) == 0) {
                *out = k.code;
                return true;
            }
        PyErr_SetObject(PyExc_KeyError, o);
        return false;
    }
    int v;
    if (!convert(o, &v, h)) return false;
    *out = (tir_dtype)v;
    return true;
}
bool convert(PyObject* o, const tir_epilogue** out, Held& h) {
    *out = nullptr;
    if (o == Py_None) return true;
    // (any object has a buffer that could be read as the struct: a bias array's first values would become its address)
    const int is = g_epilogue_type ? PyObject_IsInstance(o, g_epilogue_type) : 0;
    if (is < 0) return false;
    if (!is) {
        PyErr_Format(PyExc_TypeError, "epilogue: expected an Epilogue or None, got %.200s", Py_TYPE(o)->tp_name);
        return false;
    }
    if (PyObject_GetBuffer(o, &h.view, PyBUF_SIMPLE) != 0) return false;
    h.used = true;
    if ((size_t)h.view.len < sizeof(tir_epilogue)) {
        PyErr_SetString(PyExc_ValueError, "epilogue: the buffer is smaller than tir_epilogue");
        return false;
    }
    *out = (const tir_epilogue*)h.view.buf;
    return true;
}

template <class... A, size_t... I>
PyObject* invoke(tir_status (*fn)(A...), PyObject* const* args, std::index_sequence<I...>) {
    std::tuple<A...> v{};
    Held held;
    constexpr size_t last = sizeof...(A) - 1;
    bool ok = true;
    // (left to right, stopping at the first argument that does not convert)
    ((ok = ok && (I == last ? to_stream(args[I], (void**)&std::get<last>(v)) : convert(args[I], &std::get<I>(v), held))), ...);
    if (!ok) return nullptr;
    tir_status st;
    Py_BEGIN_ALLOW_THREADS
    st = fn(std::get<I>(v)...);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong((long)st);
}

template <class... A>
PyObject* call(tir_status (*fn)(A...), const char* name, PyObject* const* args, Py_ssize_t n) {
    static_assert(std::is_same<typename std::tuple_element<sizeof...(A) - 1, std::tuple<A...>>::type, tir_stream>::value, "the stream comes last");
    if (n != (Py_ssize_t)sizeof...(A)) {
        PyErr_Format(PyExc_TypeError, "%s takes %zd arguments (%zd given)", name, (Py_ssize_t)sizeof...(A), n);
        return nullptr;
    }
    return invoke(fn, args, std::index_sequence_for<A...>());
}

#define TIR_PY(fn) \
    PyObject* py_##fn(PyObject*, PyObject* const* args, Py_ssize_t n) { return call(&fn, #fn, args, n); }
TIR_PY(tir_gemm_fused)
TIR_PY(tir_batch_matmul_fused)
TIR_PY(tir_conv2d_fused)
TIR_PY(tir_conv1d)
TIR_PY(tir_conv3d)
TIR_PY(tir_conv2d_transpose)
TIR_PY(tir_attention)
#undef TIR_PY

// set_epilogue_type(cls): called once by the binding, before any operator.
PyObject* py_set_epilogue_type(PyObject*, PyObject* cls) {
    if (!PyType_Check(cls)) {
        PyErr_SetString(PyExc_TypeError, "set_epilogue_type: expected a class");
        return nullptr;
    }
    Py_INCREF(cls);
    Py_XSETREF(g_epilogue_type, cls);
    Py_RETURN_NONE;
}

#define TIR_METHOD(fn) {#fn, (PyCFunction)(void (*)(void))py_##fn, METH_FASTCALL, nullptr}
PyMethodDef kMethods[] = {TIR_METHOD(tir_gemm_fused), TIR_METHOD(tir_batch_matmul_fused), TIR_METHOD(tir_conv2d_fused), TIR_METHOD(tir_conv1d),
                          TIR_METHOD(tir_conv3d), TIR_METHOD(tir_conv2d_transpose), TIR_METHOD(tir_attention),
                          {"set_epilogue_type", py_set_epilogue_type, METH_O, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

PyObject* attribute(const char* module, const char* name) {
    PyObject* m = PyImport_ImportModule(module);
    if (!m) return nullptr;
    PyObject* a = PyObject_GetAttrString(m, name);
    Py_DECREF(m);
    return a;
}

}  // namespace

PyMODINIT_FUNC PyInit__native(void) {
    g_data_ptr = PyUnicode_InternFromString("data_ptr");
    g_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    g_current_stream = attribute("torch.cuda", "current_stream");
    if (g_current_stream) g_get_device = attribute("torch._C", "_cuda_getDevice");
    if (g_get_device) g_raw_stream = attribute("torch._C", "_cuda_getCurrentRawStream");
    if (!g_data_ptr || !g_cuda_stream || !g_raw_stream) return nullptr;
    return PyModule_Create(&kModule);
}
