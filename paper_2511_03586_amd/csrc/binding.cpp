// The entry points of perf.h that programs call per operator, as functions of a CPython module: positional arguments, the
// status as the result.  A call through ctypes spends 1.6 us (softmax, 10 arguments) to 2.3 us (gemm, 19) on converting
// its arguments, a fourth of what a small operator's call takes from end to end; these functions take 0.2 us.
//
// Only the plain types are converted here (None and int for addresses, int, float); anything else that ctypes takes (numpy
// integers, ctypes pointers, integers that wrap) goes to the ctypes function, which set_fallback's callable finds by name.
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
    if (n != (Py_ssize_t)sizeof...(A) || !(get(args[I], std::get<I>(a)) && ...)) {
        if (!g_fallback) {
            PyErr_SetString(PyExc_RuntimeError, "set_fallback has not been called");
            return nullptr;
        }
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

#define PERF_METHOD(F) \
    PyObject *m_##F(PyObject *, PyObject *const *args, Py_ssize_t n) { return call(#F, F, args, n); }
PERF_METHOD(perf_softmax)
PERF_METHOD(perf_layernorm)
PERF_METHOD(perf_gemm)
PERF_METHOD(perf_gemm_softmax)
PERF_METHOD(perf_conv2d)
PERF_METHOD(perf_rmsnorm)
PERF_METHOD(perf_reduce_mean)
PERF_METHOD(perf_reduce_mean_ws)
PERF_METHOD(perf_eltwise)
PERF_METHOD(perf_batchnorm)
PERF_METHOD(perf_batchnorm_static)
PERF_METHOD(perf_copy)
#undef PERF_METHOD

PyObject *set_fallback(PyObject *, PyObject *f)
{
    Py_INCREF(f);
    Py_XSETREF(g_fallback, f);
    Py_RETURN_NONE;
}

#define PERF_ENTRY(F) {#F, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(m_##F)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    PERF_ENTRY(perf_softmax), PERF_ENTRY(perf_layernorm), PERF_ENTRY(perf_gemm), PERF_ENTRY(perf_gemm_softmax),
    PERF_ENTRY(perf_conv2d), PERF_ENTRY(perf_rmsnorm), PERF_ENTRY(perf_reduce_mean), PERF_ENTRY(perf_reduce_mean_ws),
    PERF_ENTRY(perf_eltwise), PERF_ENTRY(perf_batchnorm), PERF_ENTRY(perf_batchnorm_static), PERF_ENTRY(perf_copy),
    {"set_fallback", set_fallback, METH_O, nullptr}, {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void) { return PyModule_Create(&module); }
