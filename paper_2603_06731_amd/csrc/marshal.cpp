// Argument marshalling of the Python binding: takes a call's Python objects, turns them into the C arguments of one entry point of pbk.h and
// calls it, without the interpreter.  A call that ctypes marshals costs the host some 2 us beyond the launch, and most small kernels end sooner:
// 256 x 256 x 256 in fp32, 4.9 us a call on the host, of which the launch and the choice of the kernel are the half.
//
// A function here returns None, and calls nothing, for anything but plain arguments (integers in range, floats, None, objects with data_ptr() or
// cuda_stream): the binding then goes through ctypes, whose conversions and errors are the contract.  What a data_ptr() or cuda_stream of the caller's
// raises leaves this call as it is (but AttributeError and TypeError, which an object without one gives as well): nothing of the caller's runs again after it
// has failed, and no interrupt is lost.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>
#include <limits.h>
#include <string_view>
#include <tuple>
#include <type_traits>
#include <utility>
#include "../../include/pbk.h"

namespace {

PyObject *g_data_ptr, *g_cuda_stream;            // method and attribute names

bool as_address(PyObject* o, void*& v) {
    if (!PyLong_CheckExact(o)) return false;
    const unsigned long long a = PyLong_AsUnsignedLongLong(o);
    if (a == (unsigned long long)-1 && PyErr_Occurred()) { PyErr_Clear(); return false; }
    v = (void*)(uintptr_t)a;
    return true;
}

// the address that an attribute (called: a method) of `o` gives.  False with an exception set: the caller's own
bool address_of(PyObject* o, PyObject* name, bool call, void*& v) {
    PyObject* r = call ? PyObject_CallMethodNoArgs(o, name) : PyObject_GetAttr(o, name);
    if (!r) {
        if (PyErr_ExceptionMatches(PyExc_AttributeError) || PyErr_ExceptionMatches(PyExc_TypeError)) PyErr_Clear();
        return false;
    }
    const bool ok = as_address(r, v);
    Py_DECREF(r);
    return ok;
}

template <typename T> bool get(PyObject* o, T& v) {
    if constexpr (std::is_pointer<T>::value) {
        void* a = nullptr;
        if (o != Py_None && !as_address(o, a)) {
            constexpr bool stream = std::is_same<T, hipStream_t>::value;
            if (!address_of(o, stream ? g_cuda_stream : g_data_ptr, !stream, a)) return false;
        }
        v = (T)a;
        return true;
    } else if constexpr (std::is_same<T, float>::value) {
        if (!PyFloat_CheckExact(o)) return false;
        v = (float)PyFloat_AS_DOUBLE(o);
        return true;
    } else {
        static_assert(std::is_integral<T>::value, "types of the C interface");
        if (!PyLong_Check(o)) return false;
        int over = 0;
        const long long x = PyLong_AsLongLongAndOverflow(o, &over);
        if (over || (sizeof(T) == 4 && (x < INT_MIN || x > INT_MAX))) return false;
        v = (T)x;
        return true;
    }
}

// An enum travels as the int that it is in the calling convention: any value that Python passes is for the entry point to judge.
template <typename T> struct Passed { typedef T type; };
template <> struct Passed<pbk_dtype> { typedef int type; };
template <> struct Passed<pbk_epilogue> { typedef int type; };

// ID keeps entry points of the same type apart
template <int ID, typename F> struct Call;
template <int ID, typename R, typename... A> struct Call<ID, R(A...)> {
    inline static R (*fn)(typename Passed<A>::type...) = nullptr;      // set by bind(): the library is loaded later than this module
    template <size_t... I> static PyObject* run(PyObject* const* args, std::index_sequence<I...>) {
        std::tuple<typename Passed<A>::type...> v;
        if (!(get(args[I], std::get<I>(v)) && ...)) {
            if (PyErr_Occurred()) return nullptr;
            Py_RETURN_NONE;
        }
        R r;
        Py_BEGIN_ALLOW_THREADS
        r = fn(std::get<I>(v)...);
        Py_END_ALLOW_THREADS
        return PyLong_FromLong((long)r);
    }
    static PyObject* call(PyObject*, PyObject* const* args, Py_ssize_t n) {
        if (!fn || n != (Py_ssize_t)sizeof...(A)) Py_RETURN_NONE;
        return run(args, std::make_index_sequence<sizeof...(A)>{});
    }
};

#define PBK_ENTRIES(X) X(0, pbk_matmul) X(1, pbk_batched_matmul) X(2, pbk_conv2d_nhwc) X(3, pbk_conv2d_nhwc_pad4) X(4, pbk_conv2d_transpose_nhwc) \
    X(5, pbk_matmul_residual) X(6, pbk_conv2d_nhwc_residual) X(7, pbk_matmul_int8) X(8, pbk_conv2d_nhwc_int8) X(9, pbk_matmul_int8_bn) \
    X(10, pbk_conv2d_nhwc_int8_bn) X(11, pbk_attention) X(12, pbk_attention_causal)

// bind(name, address of the loaded entry point)
PyObject* bind(PyObject*, PyObject* args) {
    const char* name;
    unsigned long long address;
    if (!PyArg_ParseTuple(args, "sK", &name, &address)) return nullptr;
    const std::string_view n = name;
#define PBK_BIND(ID, ENTRY) if (n == #ENTRY) { typedef Call<ID, decltype(ENTRY)> C; C::fn = (decltype(C::fn))(uintptr_t)address; Py_RETURN_TRUE; }
    PBK_ENTRIES(PBK_BIND)
    Py_RETURN_FALSE;
}

PyMethodDef g_methods[] = {
#define PBK_METHOD(ID, ENTRY) {#ENTRY, (PyCFunction)(void (*)(void))&Call<ID, decltype(ENTRY)>::call, METH_FASTCALL, nullptr},
    PBK_ENTRIES(PBK_METHOD)
    {"bind", &bind, METH_VARARGS, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) {
    g_data_ptr = PyUnicode_InternFromString("data_ptr");
    g_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    if (!g_data_ptr || !g_cuda_stream) return nullptr;
    return PyModule_Create(&g_module);
}
