// Argument marshalling of the Python binding for the calls of a decode step: a Python call's arguments to the
// C ABI's, without a Python function or a ctypes conversion for each.  A launch costs the runtime 2.9 us on the
// host; conversions in Python and ctypes added 2.1 us to a decode call's and 2.0 to an append's, now 0.6 and
// 0.5.  Launches that the GPU has done sooner wait for the host: appends 6.1 us a pass -> 4.8.
//   structs(shape, pool): the ctypes classes of hetis_attn_shape and hetis_kv_pool, before the first call.
//   bind(name, address) -> callable for the library function `name` at `address`; None for other names.
// The callable takes positional arguments only, as many as the C function.  By the type of the parameter:
// structs are instances of those classes (a pool may be None), pointers are None, an int, or
// an object with data_ptr() (a torch tensor) or .ctypes.data (a numpy array); numbers are converted as int()
// and float() do.  The interpreter lock is released during the call, as ctypes does.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstdint>
#include <cstring>
#include <tuple>
#include <type_traits>
#include <utility>

#include "../../include/hetis_attn.h"
#include "../../include/hetis_kv.h"

namespace {

PyObject *s_data_ptr, *s_ctypes, *s_data;      // interned attribute names
PyObject *shape_type, *pool_type;               // the binding's classes of the two structures

bool address_of(PyObject *o, void **out)
{
    if (o == Py_None) {
        *out = nullptr;
        return true;
    }
    PyObject *n = nullptr;
    if (PyLong_Check(o)) {
        Py_INCREF(o);
        n = o;
    } else {
        n = PyObject_CallMethodNoArgs(o, s_data_ptr);
        if (!n && PyErr_ExceptionMatches(PyExc_AttributeError)) {
            PyErr_Clear();
            PyObject *c = PyObject_GetAttr(o, s_ctypes);
            if (c) n = PyObject_GetAttr(c, s_data);
            Py_XDECREF(c);
        }
        if (!n) return false;
    }
    const unsigned long long v = PyLong_AsUnsignedLongLongMask(n);
    Py_DECREF(n);
    if (v == (unsigned long long)-1 && PyErr_Occurred()) return false;
    *out = reinterpret_cast<void *>((uintptr_t)v);
    return true;
}

template <class T>
bool convert(PyObject *o, T &out)
{
    if constexpr (std::is_same_v<T, float>) {
        PyObject *n = PyNumber_Float(o);
        if (!n) return false;
        out = (float)PyFloat_AS_DOUBLE(n);
        Py_DECREF(n);
        return true;
    } else if constexpr (std::is_integral_v<T>) {
        PyObject *n = PyLong_Check(o) ? (Py_INCREF(o), o) : PyNumber_Long(o);
        if (!n) return false;
        const unsigned long long v = PyLong_AsUnsignedLongLongMask(n);
        Py_DECREF(n);
        if (v == (unsigned long long)-1 && PyErr_Occurred()) return false;
        out = (T)v;
        return true;
    } else {
        using S = std::remove_cv_t<std::remove_pointer_t<T>>;
        if constexpr (std::is_same_v<S, hetis_attn_shape> || std::is_same_v<S, hetis_kv_pool>) {
            if (o == Py_None && std::is_same_v<S, hetis_kv_pool>) {      // (a shape has to be one)
                out = nullptr;
                return true;
            }
            PyObject *type = std::is_same_v<S, hetis_kv_pool> ? pool_type : shape_type;
            const int is = type ? PyObject_IsInstance(o, type) : 0;
            if (is <= 0) {
                if (is == 0) PyErr_Format(PyExc_TypeError, "a structure argument is a %s", Py_TYPE(o)->tp_name);
                return false;
            }
            Py_buffer view;
            if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) return false;
            out = static_cast<T>(view.buf);     // the caller holds the object until the call returns
            PyBuffer_Release(&view);
            return true;
        } else {
            void *a = nullptr;
            if (!address_of(o, &a)) return false;
            out = static_cast<T>(a);
            return true;
        }
    }
}

template <class F>
struct Call;
template <class... A>
struct Call<int (*)(A...)> {
    template <size_t... I>
    static PyObject *run(int (*f)(A...), PyObject *const *args, std::index_sequence<I...>)
    {
        std::tuple<A...> a{};
        if (!(convert(args[I], std::get<I>(a)) && ...)) return nullptr;
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = f(std::get<I>(a)...);
        Py_END_ALLOW_THREADS
        return PyLong_FromLong(rc);
    }
    static PyObject *entry(PyObject *self, PyObject *const *args, Py_ssize_t n)
    {
        if (n != (Py_ssize_t)sizeof...(A)) {
            PyErr_Format(PyExc_TypeError, "%zu arguments expected, %zd given", sizeof...(A), n);
            return nullptr;
        }
        auto f = reinterpret_cast<int (*)(A...)>(PyLong_AsVoidPtr(self));
        return run(f, args, std::index_sequence_for<A...>{});
    }
};

#define HETIS_CALL(name) \
    {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&Call<decltype(&name)>::entry)), METH_FASTCALL, nullptr}
PyMethodDef calls[] = {
    HETIS_CALL(hetis_attn_decode), HETIS_CALL(hetis_attn_decode_ws), HETIS_CALL(hetis_attn_decode_step),
    HETIS_CALL(hetis_attn_decode_step_ws), HETIS_CALL(hetis_attn_decode_pairs), HETIS_CALL(hetis_attn_decode_pairs_ws),
    HETIS_CALL(hetis_attn_decode_pairs_step), HETIS_CALL(hetis_attn_decode_pairs_step_ws),
    HETIS_CALL(hetis_attn_decode_split), HETIS_CALL(hetis_attn_decode_split_ws), HETIS_CALL(hetis_attn_merge),
    HETIS_CALL(hetis_kv_append), HETIS_CALL(hetis_kv_append_pairs), HETIS_CALL(hetis_kv_store),
    HETIS_CALL(hetis_kv_fetch), HETIS_CALL(hetis_kv_copy_tiles),
};

PyObject *bind(PyObject *, PyObject *args)
{
    const char *name;
    unsigned long long address;
    if (!PyArg_ParseTuple(args, "sK", &name, &address)) return nullptr;
    for (PyMethodDef &d : calls) {
        if (std::strcmp(d.ml_name, name) != 0) continue;
        PyObject *self = PyLong_FromVoidPtr(reinterpret_cast<void *>((uintptr_t)address));
        if (!self) return nullptr;
        PyObject *f = PyCFunction_New(&d, self);
        Py_DECREF(self);
        return f;
    }
    Py_RETURN_NONE;
}

PyObject *structs(PyObject *, PyObject *args)
{
    PyObject *shape, *pool;
    if (!PyArg_ParseTuple(args, "OO", &shape, &pool)) return nullptr;
    Py_INCREF(shape);
    Py_INCREF(pool);
    Py_XSETREF(shape_type, shape);
    Py_XSETREF(pool_type, pool);
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"bind", bind, METH_VARARGS, nullptr},
                         {"structs", structs, METH_VARARGS, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void)
{
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_ctypes = PyUnicode_InternFromString("ctypes");
    s_data = PyUnicode_InternFromString("data");
    if (!s_data_ptr || !s_ctypes || !s_data) return nullptr;
    shape_type = pool_type = nullptr;
    return PyModule_Create(&module);
}
