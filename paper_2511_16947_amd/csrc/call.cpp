// Marshalling of a library call from Python: call(function, kinds, stream, shape, argument, ...) -> return code.
//   function, shape   addresses
//   kinds             a character per argument: 't' a tensor or None, 'i' what ctypes takes for an int32_t: an int, a c_int32, what
//                     has __index__ (NumPy's integers, integer tensors of one element) or an _as_parameter_ of these
//   stream            what to call for the stream handle, which is passed last, once all arguments have been accepted
//
// Every argument of an entry point of finemoe.h is a pointer, an integer of at most 64 bits or a size, all of which the C calling
// convention of x86-64 passes as 64-bit integers (a narrower parameter is the low part of its slot), so that one function
// type serves them all.  A small layer is bound by the host: eight calls and twelve launches for 256 fp32 tokens on four ranks, whose
// 59 tensors went through 0.3 us of Python each, and the calls through 1 us of ctypes.
//
// A tensor is asked the same questions, in the same order, as Python code would ask it (is_cuda, is_contiguous(), data_ptr()).
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstdint>

#if !defined(__x86_64__)
#error "arguments are passed as 64-bit integers: x86-64 calling convention"
#endif

namespace {

constexpr Py_ssize_t kMaxArgs = 24;
PyObject *s_is_cuda, *s_is_contiguous, *s_data_ptr, *s_value, *s_as_parameter;
PyObject *c_int32, *refused;      // ctypes.c_int32; a ctypes.ArgumentError that is a TypeError too

bool integer(PyObject* o, uint64_t& out) {
    out = PyLong_AsUnsignedLongLongMask(o);
    return !(out == (uint64_t)-1 && PyErr_Occurred());
}

// true, false, or -1 with an exception set; takes the reference
int truth(PyObject* o) {
    if (o == nullptr) return -1;
    const int v = PyObject_IsTrue(o);
    Py_DECREF(o);
    return v;
}

bool pointer(PyObject* t, uint64_t& out) {
    int ok = truth(PyObject_GetAttr(t, s_is_cuda));
    if (ok == 1) ok = truth(PyObject_CallMethodNoArgs(t, s_is_contiguous));
    if (ok < 0) return false;
    if (ok == 0) {
        PyErr_SetString(PyExc_AssertionError, "device-resident contiguous tensors only");
        return false;
    }
    PyObject* p = PyObject_CallMethodNoArgs(t, s_data_ptr);
    if (p == nullptr) return false;
    const bool good = PyLong_Check(p) ? integer(p, out) : (PyErr_SetString(PyExc_TypeError, "data_ptr() is no integer"), false);
    Py_DECREF(p);
    return good;
}

// what is no int; argument number for the message
bool other_integer(PyObject* o, Py_ssize_t number, uint64_t& out) {
    const int simple = PyObject_IsInstance(o, c_int32);
    if (simple < 0) return false;
    PyObject* v = simple ? PyObject_GetAttr(o, s_value) : PyNumber_Index(o);
    if (v == nullptr && !simple) {
        PyErr_Clear();
        v = PyObject_GetAttr(o, s_as_parameter);
        if (v == nullptr) {
            PyErr_Clear();
            PyErr_Format(refused, "argument %zd: an integer, not %s", number, Py_TYPE(o)->tp_name);
        }
    }
    if (v == nullptr) return false;
    bool ok = false;
    if (PyLong_Check(v)) {
        ok = integer(v, out);
    } else if (Py_EnterRecursiveCall(" in an _as_parameter_") == 0) {
        ok = other_integer(v, number, out);
        Py_LeaveRecursiveCall();
    }
    Py_DECREF(v);
    return ok;
}

PyObject* call(PyObject*, PyObject* const* args, Py_ssize_t n) {
    Py_ssize_t n_args = 0;
    const char* kinds = n >= 4 ? PyUnicode_AsUTF8AndSize(args[1], &n_args) : nullptr;
    if (kinds == nullptr || n != 4 + n_args || n_args + 2 > kMaxArgs) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_TypeError, "call(function, kinds, stream, shape, an argument for each kind)");
        return nullptr;
    }
    uint64_t function, v[kMaxArgs] = {};
    if (!PyLong_Check(args[0]) || !PyLong_Check(args[3]) || !integer(args[0], function) || !integer(args[3], v[0]) || function == 0) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_TypeError, "addresses of the function and of the shape");
        return nullptr;
    }
    for (Py_ssize_t i = 0; i < n_args; ++i) {
        PyObject* o = args[4 + i];
        if (kinds[i] == 't') {
            if (o != Py_None && !pointer(o, v[1 + i])) return nullptr;
        } else if (!(PyLong_Check(o) ? integer(o, v[1 + i]) : other_integer(o, i + 1, v[1 + i]))) {
            return nullptr;
        }
    }
    PyObject* handle = PyObject_CallNoArgs(args[2]);
    if (handle == nullptr) return nullptr;
    const bool ok = PyLong_Check(handle) ? integer(handle, v[1 + n_args]) : (PyErr_SetString(PyExc_TypeError, "stream handle"), false);
    Py_DECREF(handle);
    if (!ok) return nullptr;
    using U = uint64_t;
    using Fn = int (*)(U, U, U, U, U, U, U, U, U, U, U, U, U, U, U, U, U, U, U, U, U, U, U, U);
    const Fn f = reinterpret_cast<Fn>(function);
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f(v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7], v[8], v[9], v[10], v[11], v[12], v[13], v[14], v[15], v[16], v[17],
           v[18], v[19], v[20], v[21], v[22], v[23]);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

PyMethodDef methods[] = {
    {"call", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(call)), METH_FASTCALL, "call(function, kinds, stream, shape, ...) -> return code"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__call() {
    s_is_cuda = PyUnicode_InternFromString("is_cuda");
    s_is_contiguous = PyUnicode_InternFromString("is_contiguous");
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_value = PyUnicode_InternFromString("value");
    s_as_parameter = PyUnicode_InternFromString("_as_parameter_");
    if (!s_is_cuda || !s_is_contiguous || !s_data_ptr || !s_value || !s_as_parameter) return nullptr;
    PyObject* ctypes = PyImport_ImportModule("ctypes");
    if (ctypes == nullptr) return nullptr;
    c_int32 = PyObject_GetAttrString(ctypes, "c_int32");
    PyObject* base = PyObject_GetAttrString(ctypes, "ArgumentError");
    Py_DECREF(ctypes);
    if (c_int32 == nullptr || base == nullptr) return nullptr;
    PyObject* bases = PyTuple_Pack(2, base, PyExc_TypeError);
    Py_DECREF(base);
    if (bases == nullptr) return nullptr;
    refused = PyErr_NewException("paper_2511_16947_amd.ArgumentError", bases, nullptr);
    Py_DECREF(bases);
    if (refused == nullptr) return nullptr;
    return PyModule_Create(&module);
}
