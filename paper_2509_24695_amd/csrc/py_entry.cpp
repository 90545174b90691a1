// CPython calls of the C ABI's launching entry points: turns Python arguments into C ones and calls the function.  The ctypes
// route took 3.7 to 4.5 us per call for this (structures and pointer objects made anew, eleven conversions), more than the
// launch itself; small calls waited for it (layer of 2 heads, 1 024 tokens: 14.7 us for two launches whose kernels take 11).
// The functions are looked up in the library that binding.py has loaded; nothing is linked.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <dlfcn.h>

#include <tuple>
#include <utility>

#include "../../include/sv_linattn.h"
#include "../../include/sv_tconv.h"

namespace {

PyObject *g_argument_error;       // ctypes.ArgumentError, what a wrong argument has always raised

struct Names {
    PyObject *data_ptr, *cuda_stream, *numel, *element_size;
    PyObject *B, *H, *N, *d, *stride_b, *stride_h, *stride_n, *dtype;
    PyObject *frames, *rows, *cols, *n_t, *n_h, *n_w, *cs_t, *cs_h, *cs_w;
} g;

bool to_i64(PyObject *o, int64_t &out)          // whole numbers; bits above the C type are dropped
{
    if (PyFloat_Check(o)) {
        PyErr_SetString(PyExc_TypeError, "int expected instead of float");
        return false;
    }
    PyObject *n = PyLong_Check(o) ? (Py_INCREF(o), o) : PyNumber_Index(o);
    if (!n) return false;
    out = (int64_t)PyLong_AsUnsignedLongLongMask(n);
    Py_DECREF(n);
    return !PyErr_Occurred();
}
template <typename T> bool attr_int(PyObject *o, PyObject *name, T &out)
{
    PyObject *v = PyObject_GetAttr(o, name);
    int64_t x = 0;
    const bool ok = v && to_i64(v, x);
    Py_XDECREF(v);
    out = (T)x;
    return ok;
}
// Device address of a tensor, or an integer address / None as given.
bool to_ptr(PyObject *o, void *&out)
{
    out = nullptr;
    if (o == Py_None) return true;
    int64_t x = 0;
    if (PyLong_Check(o)) {
        if (!to_i64(o, x)) return false;
    } else {
        PyObject *v = PyObject_CallMethodNoArgs(o, g.data_ptr);
        const bool ok = v && to_i64(v, x);
        Py_XDECREF(v);
        if (!ok) return false;
    }
    out = reinterpret_cast<void *>(x);
    return true;
}
bool attr_ptr(PyObject *o, PyObject *name, const float *&out)
{
    PyObject *v = PyObject_GetAttr(o, name);
    void *p = nullptr;
    const bool ok = v && to_ptr(v, p);
    Py_XDECREF(v);
    out = static_cast<const float *>(p);
    return ok;
}

// One kind of argument each: holds the C value, get() fills it from args[i].
struct Ptr {
    void *v;
    bool get(PyObject *const *args, int i) { return to_ptr(args[i], v); }
    void *c() { return v; }
};
struct Desc {
    sv_tensor_desc v;
    bool present;
    bool get(PyObject *const *args, int i)
    {
        PyObject *o = args[i];
        present = o != Py_None;
        return !present || (attr_int(o, g.B, v.B) && attr_int(o, g.H, v.H) && attr_int(o, g.N, v.N) && attr_int(o, g.d, v.d) &&
                            attr_int(o, g.stride_b, v.stride_b) && attr_int(o, g.stride_h, v.stride_h) &&
                            attr_int(o, g.stride_n, v.stride_n) && attr_int(o, g.dtype, v.dtype));
    }
    const sv_tensor_desc *c() { return present ? &v : nullptr; }
};
struct Rope {
    sv_rope3d v;
    bool present;
    bool get(PyObject *const *args, int i)
    {
        PyObject *o = args[i];
        present = o != Py_None;
        return !present || (attr_int(o, g.frames, v.frames) && attr_int(o, g.rows, v.rows) && attr_int(o, g.cols, v.cols) &&
                            attr_int(o, g.n_t, v.n_t) && attr_int(o, g.n_h, v.n_h) && attr_int(o, g.n_w, v.n_w) &&
                            attr_ptr(o, g.cs_t, v.cs_t) && attr_ptr(o, g.cs_h, v.cs_h) && attr_ptr(o, g.cs_w, v.cs_w));
    }
    const sv_rope3d *c() { return present ? &v : nullptr; }
};
struct Int {                           // an index or size, as a 32-bit integer
    int32_t v;
    bool get(PyObject *const *args, int i)
    {
        int64_t x = 0;
        if (!to_i64(args[i], x)) {
            if (PyErr_ExceptionMatches(PyExc_TypeError)) {
                PyErr_Clear();
                PyErr_Format(g_argument_error, "argument %d: <class 'TypeError'>: wrong type", i + 1);
            }
            return false;
        }
        v = (int32_t)x;
        return true;
    }
    int32_t c() { return v; }
};
struct Flag {                          // int(x)
    int32_t v;
    bool get(PyObject *const *args, int i)
    {
        PyObject *n = PyNumber_Long(args[i]);
        int64_t x = 0;
        const bool ok = n && to_i64(n, x);
        Py_XDECREF(n);
        v = (int32_t)x;
        return ok;
    }
    int32_t c() { return v; }
};
struct Eps {                           // float(x)
    float v;
    bool get(PyObject *const *args, int i)
    {
        PyObject *f = PyNumber_Float(args[i]);
        if (f) v = (float)PyFloat_AS_DOUBLE(f);
        Py_XDECREF(f);
        return f != nullptr;
    }
    float c() { return v; }
};
struct Bytes {                         // size of the workspace in the argument before; None: that of the tensor
    size_t v;
    bool get(PyObject *const *args, int i)
    {
        int64_t x = 0, e = 1;
        if (args[i] != Py_None) {
            PyObject *n = PyNumber_Long(args[i]);
            const bool ok = n && to_i64(n, x);
            Py_XDECREF(n);
            if (!ok) return false;
        } else {
            PyObject *n = PyObject_CallMethodNoArgs(args[i - 1], g.numel);
            PyObject *s = n ? PyObject_CallMethodNoArgs(args[i - 1], g.element_size) : nullptr;
            const bool ok = s && to_i64(n, x) && to_i64(s, e);
            Py_XDECREF(n);
            Py_XDECREF(s);
            if (!ok) return false;
        }
        v = (size_t)(x * e);
        return true;
    }
    size_t c() { return v; }
};
struct Stream {                        // a stream object, an integer handle, or None
    void *v;
    bool get(PyObject *const *args, int i)
    {
        v = nullptr;
        if (args[i] == Py_None) return true;
        int64_t x = 0;
        if (PyLong_Check(args[i])) {
            if (!to_i64(args[i], x)) return false;
        } else if (!attr_int(args[i], g.cuda_stream, x)) {
            return false;
        }
        v = reinterpret_cast<void *>(x);
        return true;
    }
    void *c() { return v; }
};

template <class Fn, class... A, size_t... I>
PyObject *call(Fn fn, const char *name, PyObject *const *args, Py_ssize_t n, std::tuple<A...> a, std::index_sequence<I...>)
{
    if (!fn || n != (Py_ssize_t)sizeof...(A)) {
        PyErr_Format(PyExc_TypeError, fn ? "%s: takes %d arguments" : "%s: the library is not attached (%d arguments)", name, (int)sizeof...(A));
        return nullptr;
    }
    if (!(std::get<I>(a).get(args, (int)I) && ...)) return nullptr;
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = (int)fn(static_cast<decltype(std::get<I>(a).c())>(std::get<I>(a).c())...);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

// void * to the typed pointers that the C declarations have
struct AnyPtr {
    void *p;
    template <class T> operator T *() const { return static_cast<T *>(p); }
};
struct TypedPtr : Ptr {
    AnyPtr c() { return AnyPtr{v}; }
};

#define ENTRY(NAME, ...)                                                                                             \
    decltype(&NAME) p_##NAME;                                                                                        \
    PyObject *py_##NAME(PyObject *, PyObject *const *args, Py_ssize_t n)                                             \
    {                                                                                                                \
        using Args = std::tuple<__VA_ARGS__>;                                                                        \
        return call(p_##NAME, #NAME, args, n, Args{}, std::make_index_sequence<std::tuple_size<Args>::value>());     \
    }
using P = TypedPtr;
ENTRY(sv_linattn_state, P, P, Desc, Int, Int, Flag, P, P, P, Bytes, Stream)
ENTRY(sv_linattn_apply, P, Desc, Int, Int, P, P, Eps, P, Stream)
ENTRY(sv_block_linattn_step, P, P, P, Desc, P, P, Eps, P, P, Bytes, Stream)
ENTRY(sv_block_linattn_lookahead, P, P, P, Desc, P, P, Eps, P, P, Bytes, Stream)
ENTRY(sv_block_linattn_step_static, P, P, P, Desc, P, P, Eps, P, Stream)
ENTRY(sv_linattn_state_rope, P, P, Desc, P, Int, Int, Flag, P, P, P, Bytes, Stream)
ENTRY(sv_linattn_apply_rope, P, Desc, P, Int, Int, P, P, Eps, P, Stream)
ENTRY(sv_block_linattn_step_rope, P, P, P, Desc, P, P, P, Eps, P, P, Bytes, Stream)
ENTRY(sv_block_linattn_lookahead_rope, P, P, P, Desc, P, P, P, Eps, P, P, Bytes, Stream)
ENTRY(sv_linattn_state_rope3d, P, P, Desc, Rope, Int, Int, Flag, P, P, P, Bytes, Stream)
ENTRY(sv_linattn_apply_rope3d, P, Desc, Rope, Int, Int, P, P, Eps, P, Stream)
ENTRY(sv_block_linattn_step_rope3d, P, P, P, Desc, Rope, P, P, Eps, P, P, Bytes, Stream)
ENTRY(sv_block_linattn_lookahead_rope3d, P, P, P, Desc, Rope, P, P, Eps, P, P, Bytes, Stream)
ENTRY(sv_tconv_block_step, P, P, P, P, P, Int, Int, Int, Int, Int, Stream)

// attach(handle): the entry points of the loaded library with this dlopen handle.
PyObject *attach(PyObject *, PyObject *handle)
{
    void *lib = PyLong_AsVoidPtr(handle);
    if (!lib) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null library handle");
        return nullptr;
    }
#define ATTACH(NAME)                                                                             \
    p_##NAME = reinterpret_cast<decltype(p_##NAME)>(dlsym(lib, #NAME));                          \
    if (!p_##NAME) {                                                                             \
        PyErr_SetString(PyExc_ImportError, "the library does not export " #NAME);                \
        return nullptr;                                                                          \
    }
#define EACH(X)                                                                                                        \
    X(sv_linattn_state) X(sv_linattn_apply) X(sv_block_linattn_step) X(sv_block_linattn_lookahead)                     \
    X(sv_block_linattn_step_static) X(sv_linattn_state_rope) X(sv_linattn_apply_rope) X(sv_block_linattn_step_rope)    \
    X(sv_block_linattn_lookahead_rope) X(sv_linattn_state_rope3d) X(sv_linattn_apply_rope3d)                           \
    X(sv_block_linattn_step_rope3d) X(sv_block_linattn_lookahead_rope3d) X(sv_tconv_block_step)
    EACH(ATTACH)
    Py_RETURN_NONE;
}

#define METHOD(NAME) {#NAME, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_##NAME)), METH_FASTCALL, nullptr},
PyMethodDef methods[] = {EACH(METHOD){"attach", attach, METH_O, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_sventry", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__sventry(void)
{
#define NAME(X) if (!(g.X = PyUnicode_InternFromString(#X))) return nullptr;
    NAME(data_ptr) NAME(cuda_stream) NAME(numel) NAME(element_size)
    NAME(B) NAME(H) NAME(N) NAME(d) NAME(stride_b) NAME(stride_h) NAME(stride_n) NAME(dtype)
    NAME(frames) NAME(rows) NAME(cols) NAME(n_t) NAME(n_h) NAME(n_w) NAME(cs_t) NAME(cs_h) NAME(cs_w)
    PyObject *ctypes = PyImport_ImportModule("ctypes");
    if (!ctypes) return nullptr;
    g_argument_error = PyObject_GetAttrString(ctypes, "ArgumentError");
    Py_DECREF(ctypes);
    if (!g_argument_error) return nullptr;
    return PyModule_Create(&module_def);
}
