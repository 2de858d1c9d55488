// The entry points of perf.h that programs call per operator, as functions of a CPython module: positional arguments, the
// status as the result.  A call through ctypes spends 1.6 us (softmax, 10 arguments) to 2.3 us (gemm, 19) on converting
// its arguments, a fourth of what a small operator's call takes from end to end; these functions take 0.2 us.
//
// The module is not linked with the library: bind() takes the operators' addresses from the library that the package has
// loaded, wherever that lies.
//
// Only the plain types are converted here (None and int for addresses, int, float); anything else that ctypes takes (numpy
// integers, ctypes pointers, integers that wrap) goes to the ctypes function, which bind()'s callable finds by name.
// The call itself runs without the interpreter's lock, as through ctypes.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>
#include <tuple>
#include <type_traits>
#include <utility>
#include "../../include/perf.h"

namespace {

PyObject *g_fallback = nullptr;

template <typename T>
bool get(PyObject *o, T &out)
{
    if constexpr (std::is_pointer_v<T>) {
        if (o == Py_None) {
            out = nullptr;
            return true;
        }
        if (!PyLong_CheckExact(o)) return false;
        const unsigned long long v = PyLong_AsUnsignedLongLong(o);
        if (v == (unsigned long long)-1 && PyErr_Occurred()) {
            PyErr_Clear();
            return false;
        }
        out = reinterpret_cast<T>(static_cast<uintptr_t>(v));
        return true;
    } else if constexpr (std::is_floating_point_v<T>) {
        if (!PyFloat_CheckExact(o)) return false;
        out = (T)PyFloat_AS_DOUBLE(o);
        return true;
    } else {
        if (!PyLong_CheckExact(o)) return false;
        int overflow = 0;
        const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
        if (overflow != 0 || (sizeof(T) == 4 && v != (long long)(int)v)) return false;
        out = (T)v;
        return true;
    }
}

template <typename... A, size_t... I>
PyObject *call(const char *name, perf_status (*f)(A...), PyObject *const *args, Py_ssize_t n, std::index_sequence<I...>)
{
    std::tuple<A...> a;
    if (!g_fallback) {
        PyErr_SetString(PyExc_RuntimeError, "bind has not been called");
        return nullptr;
    }
    if (n != (Py_ssize_t)sizeof...(A) || !(get(args[I], std::get<I>(a)) && ...)) {
        PyObject *slow = PyObject_CallFunction(g_fallback, "s", name);
        if (!slow) return nullptr;
        PyObject *r = PyObject_Vectorcall(slow, args, (size_t)n, nullptr);
        Py_DECREF(slow);
        return r;
    }
    perf_status status;
    Py_BEGIN_ALLOW_THREADS
    status = f(std::get<I>(a)...);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong((long)status);
}

template <typename... A>
PyObject *call(const char *name, perf_status (*f)(A...), PyObject *const *args, Py_ssize_t n)
{
    return call(name, f, args, n, std::index_sequence_for<A...>{});
}

#define PERF_OPERATORS(X)                                                                                                        \
    X(perf_softmax) X(perf_layernorm) X(perf_gemm) X(perf_gemm_softmax) X(perf_conv2d) X(perf_rmsnorm) X(perf_reduce_mean)       \
    X(perf_reduce_mean_ws) X(perf_eltwise) X(perf_batchnorm) X(perf_batchnorm_static) X(perf_copy)

#define PERF_METHOD(F)            \
    decltype(&F) p_##F = nullptr; \
    PyObject *m_##F(PyObject *, PyObject *const *args, Py_ssize_t n) { return call(#F, p_##F, args, n); }
PERF_OPERATORS(PERF_METHOD)
#undef PERF_METHOD

// bind(address_of, fallback): address_of(name) is the address of an operator, fallback(name) its ctypes function.
PyObject *bind(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != 2) {
        PyErr_SetString(PyExc_TypeError, "bind(address_of, fallback)");
        return nullptr;
    }
    bool ok = true;
    auto set = [&](const char *name, auto &to) {
        PyObject *o = ok ? PyObject_CallFunction(args[0], "s", name) : nullptr;
        const size_t v = o ? PyLong_AsSize_t(o) : 0;
        ok = o && !PyErr_Occurred();
        Py_XDECREF(o);
        if (ok) to = reinterpret_cast<std::remove_reference_t<decltype(to)>>(v);
    };
#define PERF_SET(F) set(#F, p_##F);
    PERF_OPERATORS(PERF_SET)
#undef PERF_SET
    if (!ok) return nullptr;
    Py_INCREF(args[1]);
    Py_XSETREF(g_fallback, args[1]);
    Py_RETURN_NONE;
}

#define PERF_FAST(F, M) {#F, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(M)), METH_FASTCALL, nullptr}
#define PERF_ENTRY(F) PERF_FAST(F, m_##F),
PyMethodDef methods[] = {PERF_OPERATORS(PERF_ENTRY) PERF_FAST(bind, bind), {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void) { return PyModule_Create(&module); }
