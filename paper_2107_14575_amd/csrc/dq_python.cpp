// The Python side of the per-iteration entry points: takes the tensors' addresses, strides and row counts and calls the C
// functions of dq.h, without the GIL.  The functions are those of the library that binding.py has opened, which hands their addresses over
// (bind): the module itself needs no libdq.so, so it cannot come by another one on the loader's search path or of another copy of the
// package, whose plans have another form.  Arguments are converted as ctypes
// converts them: plain numbers here, and whatever else it takes (numpy's and torch's numbers, instances of the C types, objects with
// _as_parameter_) or refuses (ctypes.ArgumentError) by ctypes itself.  Returns the status; binding.py has the names, defaults and checks.
//
// A small call is its launch (2.6 us of HIP) and what leads there.  Through ctypes, with the attributes read in Python:
// quantize_pack 5.5 us, norm 4.8, select_bits 2.0; here 4.6, 4.1, 0.4.  An iteration of 4096 values, M = 8, 33.8 -> 28.9 us, of 2^20, M = 4,
// 35.9 -> 31.9.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <stdint.h>

#include "dq.h"

namespace {

#define DQ_FUNCTIONS(X) \
    X(dq_norm) X(dq_norm_linf) X(dq_quantize_pack) X(dq_quantize_pack_v) X(dq_norm_quantize_pack) X(dq_norm_bracket) \
    X(dq_norm_quantize_pack_bracketed) X(dq_norm_quantize_pack_bracketed_v) X(dq_unpack_dequant_reduce) X(dq_unpack_dequant_reduce_v) \
    X(dq_unpack_dequant_reduce_update) X(dq_unpack_dequant_reduce_update_v) X(dq_sign_pack) X(dq_sign_reduce) X(dq_sign_majority) \
    X(dq_select_bits) X(dq_select_bits_linf) X(dq_packed_bytes)

enum { INT32, UINT32, INT64, UINT64, ADDRESS, FLOAT32, FLOAT64, N_KINDS };

// Of one module object: copies of the package that share this file are bound each to their own library.
struct state {
#define X(fn) decltype(&::fn) fn;
    DQ_FUNCTIONS(X)
#undef X
    bool bound;
    PyObject* convert[N_KINDS]; // ctypes functions of one argument, which they return
    PyObject *data_ptr, *stride, *size, *shape, *zero;
};
state* state_of(PyObject* module) { return static_cast<state*>(PyModule_GetState(module)); }

// One call's arguments, taken one after the other; `ok` goes false with a Python exception set.
struct taker {
    const state* lib;
    PyObject* const* args;
    Py_ssize_t at = 0;
    bool ok = true;

    taker(PyObject* module, PyObject* const* a, Py_ssize_t have, Py_ssize_t want) : lib(state_of(module)), args(a)
    {
        if (!lib->bound) {
            PyErr_SetString(PyExc_RuntimeError, "no library bound");
            ok = false;
        } else if (have != want) {
            PyErr_Format(PyExc_TypeError, "%zd arguments, not %zd", want, have);
            ok = false;
        }
    }
    PyObject* converted(int kind, PyObject* o) // as ctypes passes it; a new reference
    {
        PyObject* value = PyObject_CallOneArg(lib->convert[kind], o);
        if (!value) ok = false;
        return value;
    }
    uint64_t bits_of(int kind, PyObject* o)
    {
        if (PyLong_Check(o)) return PyLong_AsUnsignedLongLongMask(o); // no error: an int
        PyObject* value = converted(kind, o);
        if (!value) return 0;
        const uint64_t v = PyLong_AsUnsignedLongLongMask(value);
        Py_DECREF(value);
        return v;
    }
    int64_t int_of(PyObject* o) // int(o); takes the reference
    {
        if (o && !PyLong_Check(o)) {
            PyObject* value = PyNumber_Long(o);
            Py_DECREF(o);
            o = value;
        }
        if (!o) {
            ok = false;
            return 0;
        }
        const uint64_t v = PyLong_AsUnsignedLongLongMask(o);
        Py_DECREF(o);
        return static_cast<int64_t>(v);
    }
    uint64_t whole(int kind) { return ok ? bits_of(kind, args[at++]) : 0; }
    int as_int() { return static_cast<int>(whole(INT32)); }
    uint32_t as_u32() { return static_cast<uint32_t>(whole(UINT32)); }
    int64_t as_i64() { return static_cast<int64_t>(whole(INT64)); }
    uint64_t as_u64() { return whole(UINT64); }
    void* address() { return reinterpret_cast<void*>(whole(ADDRESS)); } // a handle or stream
    double real(int kind)
    {
        if (!ok) return 0.0;
        PyObject* o = args[at++];
        if (PyFloat_Check(o)) return PyFloat_AS_DOUBLE(o);
        PyObject* value = converted(kind, o);
        if (!value) return 0.0;
        const double v = PyFloat_AsDouble(value);
        Py_DECREF(value);
        return v;
    }
    float as_float() { return static_cast<float>(real(FLOAT32)); }
    double as_double() { return real(FLOAT64); }
    PyObject* object() { return ok ? args[at++] : nullptr; }
    template <typename T>
    T* data_of(PyObject* t) // NULL for None
    {
        if (!ok || t == Py_None) return nullptr;
        PyObject* at_address = PyObject_CallMethodNoArgs(t, lib->data_ptr);
        if (!at_address) {
            ok = false;
            return nullptr;
        }
        const uint64_t v = bits_of(ADDRESS, at_address);
        Py_DECREF(at_address);
        return reinterpret_cast<T*>(v);
    }
    template <typename T>
    T* data()
    {
        PyObject* t = object();
        if (ok && t == Py_None) { // as None.data_ptr()
            PyErr_SetString(PyExc_AttributeError, "'NoneType' object has no attribute 'data_ptr'");
            ok = false;
        }
        return data_of<T>(t);
    }
    template <typename T>
    T* data_or_null()
    {
        return data_of<T>(object());
    }
    int64_t stride0(PyObject* t) { return ok ? int_of(PyObject_CallMethodOneArg(t, lib->stride, lib->zero)) : 0; }
    int rows(PyObject* t)
    {
        if (!ok) return 0;
        if (PyObject* size = PyObject_CallMethodOneArg(t, lib->size, lib->zero)) return static_cast<int>(int_of(size));
        if (!PyErr_ExceptionMatches(PyExc_Exception)) {
            ok = false;
            return 0;
        }
        PyErr_Clear(); // no size(0), as a tensor has: shape[0]
        PyObject* shape = PyObject_GetAttr(t, lib->shape);
        PyObject* first = shape ? PyObject_GetItem(shape, lib->zero) : nullptr;
        Py_XDECREF(shape);
        return static_cast<int>(int_of(first));
    }
};

template <typename F>
PyObject* status_of(const taker& a, F&& call)
{
    if (!a.ok) return nullptr;
    int status;
    Py_BEGIN_ALLOW_THREADS;
    status = call();
    Py_END_ALLOW_THREADS;
    return PyLong_FromLong(status);
}

template <typename T>
struct matrix { // a tensor of one row per worker
    T* data;
    int64_t stride;
    int rows;
};
template <typename T>
matrix<T> take_matrix(taker& a)
{
    PyObject* t = a.object();
    matrix<T> m = {};
    if (!a.ok) return m;
    m.rows = a.rows(t);
    m.stride = a.stride0(t);
    m.data = a.data_of<T>(t);
    return m;
}

using args_t = PyObject* const*;

// (plan, grads, norms, workspace, linf, stream)
PyObject* py_norm(PyObject* module, args_t args, Py_ssize_t n)
{
    taker a(module, args, n, 6);
    const auto* plan = static_cast<const dq_plan_t*>(a.address());
    const auto grads = take_matrix<const float>(a);
    float* norms = a.data<float>();
    void* workspace = a.data<void>();
    const int linf = a.as_int();
    void* stream = a.address();
    return status_of(a, [&] {
        return linf ? a.lib->dq_norm_linf(plan, grads.data, grads.stride, grads.rows, norms, workspace, stream)
                    : a.lib->dq_norm(plan, grads.data, grads.stride, grads.rows, norms, workspace, stream);
    });
}

// (plan, grads, norms, b, seed, step, worker_base, packed, stream)
PyObject* py_quantize_pack(PyObject* module, args_t args, Py_ssize_t n)
{
    taker a(module, args, n, 9);
    const auto* plan = static_cast<const dq_plan_t*>(a.address());
    const auto grads = take_matrix<const float>(a);
    const float* norms = a.data<const float>();
    const int b = a.as_int();
    const uint64_t seed = a.as_u64();
    const uint32_t step = a.as_u32(), worker_base = a.as_u32();
    PyObject* out = a.object();
    uint8_t* packed = a.data_of<uint8_t>(out);
    const int64_t stride = a.stride0(out);
    void* stream = a.address();
    return status_of(a, [&] {
        return a.lib->dq_quantize_pack(plan, grads.data, grads.stride, grads.rows, norms, b, seed, step, worker_base, packed, stride, stream);
    });
}

// (plan, widths, grads, norms, seed, step, worker_base, packed, stream)
PyObject* py_quantize_pack_v(PyObject* module, args_t args, Py_ssize_t n)
{
    taker a(module, args, n, 9);
    const auto* plan = static_cast<const dq_plan_t*>(a.address());
    const auto* widths = static_cast<const dq_widths_t*>(a.address());
    const auto grads = take_matrix<const float>(a);
    const float* norms = a.data<const float>();
    const uint64_t seed = a.as_u64();
    const uint32_t step = a.as_u32(), worker_base = a.as_u32();
    PyObject* out = a.object();
    uint8_t* packed = a.data_of<uint8_t>(out);
    const int64_t stride = a.stride0(out);
    void* stream = a.address();
    return status_of(a, [&] {
        return a.lib->dq_quantize_pack_v(plan, widths, grads.data, grads.stride, grads.rows, norms, seed, step, worker_base, packed, stride,
                                  stream);
    });
}

// (plan, grads, b, seed, step, worker_base, norms, packed, linf, stream)
PyObject* py_norm_quantize_pack(PyObject* module, args_t args, Py_ssize_t n)
{
    taker a(module, args, n, 10);
    const auto* plan = static_cast<const dq_plan_t*>(a.address());
    const auto grads = take_matrix<const float>(a);
    const int b = a.as_int();
    const uint64_t seed = a.as_u64();
    const uint32_t step = a.as_u32(), worker_base = a.as_u32();
    float* norms = a.data<float>();
    PyObject* out = a.object();
    uint8_t* packed = a.data_of<uint8_t>(out);
    const int64_t stride = a.stride0(out);
    const int linf = a.as_int();
    void* stream = a.address();
    return status_of(a, [&] {
        return a.lib->dq_norm_quantize_pack(plan, grads.data, grads.stride, grads.rows, linf, b, seed, step, worker_base, norms, packed, stride,
                                     stream);
    });
}

// (norms, numel, margin, lo, hi, stream)
PyObject* py_norm_bracket(PyObject* module, args_t args, Py_ssize_t n)
{
    taker a(module, args, n, 6);
    const float* norms = a.data<const float>();
    const int64_t count = a.as_i64();
    const float margin = a.as_float();
    float *lo = a.data<float>(), *hi = a.data<float>();
    void* stream = a.address();
    return status_of(a, [&] { return a.lib->dq_norm_bracket(norms, count, margin, lo, hi, stream); });
}

// (plan, widths or 0, grads, lo, hi, b, seed, step, worker_base, norms, packed, workspace, stats, linf, stream)
PyObject* py_bracketed(PyObject* module, args_t args, Py_ssize_t n)
{
    taker a(module, args, n, 15);
    const auto* plan = static_cast<const dq_plan_t*>(a.address());
    const auto* widths = static_cast<const dq_widths_t*>(a.address());
    const auto grads = take_matrix<const float>(a);
    const float *lo = a.data<const float>(), *hi = a.data<const float>();
    const int b = a.as_int();
    const uint64_t seed = a.as_u64();
    const uint32_t step = a.as_u32(), worker_base = a.as_u32();
    float* norms = a.data<float>();
    PyObject* out = a.object();
    uint8_t* packed = a.data_of<uint8_t>(out);
    const int64_t stride = a.stride0(out);
    void* workspace = a.data<void>();
    auto* stats = a.data_or_null<int64_t>();
    const int linf = a.as_int();
    void* stream = a.address();
    return status_of(a, [&] {
        return widths ? a.lib->dq_norm_quantize_pack_bracketed_v(plan, widths, grads.data, grads.stride, grads.rows, linf, lo, hi, seed, step,
                                                          worker_base, norms, packed, stride, workspace, stats, stream)
                      : a.lib->dq_norm_quantize_pack_bracketed(plan, grads.data, grads.stride, grads.rows, linf, lo, hi, b, seed, step,
                                                        worker_base, norms, packed, stride, workspace, stats, stream);
    });
}

// (plan, packed, norms, b, out, stream)
PyObject* py_reduce(PyObject* module, args_t args, Py_ssize_t n)
{
    taker a(module, args, n, 6);
    const auto* plan = static_cast<const dq_plan_t*>(a.address());
    const auto packed = take_matrix<const uint8_t>(a);
    const float* norms = a.data<const float>();
    const int b = a.as_int();
    float* out = a.data<float>();
    void* stream = a.address();
    return status_of(a, [&] { return a.lib->dq_unpack_dequant_reduce(plan, packed.data, packed.stride, packed.rows, norms, b, out, stream); });
}

// (plan, packed, norms, b, eta, x, ghat, stream)
PyObject* py_reduce_update(PyObject* module, args_t args, Py_ssize_t n)
{
    taker a(module, args, n, 8);
    const auto* plan = static_cast<const dq_plan_t*>(a.address());
    const auto packed = take_matrix<const uint8_t>(a);
    const float* norms = a.data<const float>();
    const int b = a.as_int();
    const float eta = a.as_float();
    float *x = a.data<float>(), *ghat = a.data_or_null<float>();
    void* stream = a.address();
    return status_of(a, [&] {
        return a.lib->dq_unpack_dequant_reduce_update(plan, packed.data, packed.stride, packed.rows, norms, b, eta, x, ghat, stream);
    });
}

// (plan, widths, packed, norms, out, stream)
PyObject* py_reduce_v(PyObject* module, args_t args, Py_ssize_t n)
{
    taker a(module, args, n, 6);
    const auto* plan = static_cast<const dq_plan_t*>(a.address());
    const auto* widths = static_cast<const dq_widths_t*>(a.address());
    const auto packed = take_matrix<const uint8_t>(a);
    const float* norms = a.data<const float>();
    float* out = a.data<float>();
    void* stream = a.address();
    return status_of(a, [&] { return a.lib->dq_unpack_dequant_reduce_v(plan, widths, packed.data, packed.stride, packed.rows, norms, out, stream); });
}

// (plan, widths, packed, norms, eta, x, ghat, stream)
PyObject* py_reduce_update_v(PyObject* module, args_t args, Py_ssize_t n)
{
    taker a(module, args, n, 8);
    const auto* plan = static_cast<const dq_plan_t*>(a.address());
    const auto* widths = static_cast<const dq_widths_t*>(a.address());
    const auto packed = take_matrix<const uint8_t>(a);
    const float* norms = a.data<const float>();
    const float eta = a.as_float();
    float *x = a.data<float>(), *ghat = a.data_or_null<float>();
    void* stream = a.address();
    return status_of(a, [&] {
        return a.lib->dq_unpack_dequant_reduce_update_v(plan, widths, packed.data, packed.stride, packed.rows, norms, eta, x, ghat, stream);
    });
}

// (plan, grads, packed, stream)
PyObject* py_sign_pack(PyObject* module, args_t args, Py_ssize_t n)
{
    taker a(module, args, n, 4);
    const auto* plan = static_cast<const dq_plan_t*>(a.address());
    const auto grads = take_matrix<const float>(a);
    PyObject* out = a.object();
    uint8_t* packed = a.data_of<uint8_t>(out);
    const int64_t stride = a.stride0(out);
    void* stream = a.address();
    return status_of(a, [&] { return a.lib->dq_sign_pack(plan, grads.data, grads.stride, grads.rows, packed, stride, stream); });
}

// (plan, packed, scales, out, majority, stream)
PyObject* py_sign_reduce(PyObject* module, args_t args, Py_ssize_t n)
{
    taker a(module, args, n, 6);
    const auto* plan = static_cast<const dq_plan_t*>(a.address());
    const auto packed = take_matrix<const uint8_t>(a);
    const float* scales = a.data_or_null<const float>();
    float* out = a.data<float>();
    const int majority = a.as_int();
    void* stream = a.address();
    return status_of(a, [&] {
        return majority ? a.lib->dq_sign_majority(plan, packed.data, packed.stride, packed.rows, out, stream)
                        : a.lib->dq_sign_reduce(plan, packed.data, packed.stride, packed.rows, scales, out, stream);
    });
}

// (norms: C-contiguous float32 [M][n_seg], t, T, eps_hat_q, alpha, b_min, b_max, linf) -> (status, b, Gbar)
PyObject* py_select_bits(PyObject* module, args_t args, Py_ssize_t n)
{
    taker a(module, args, n, 8);
    PyObject* array = a.object();
    const int64_t t = a.as_i64(), T = a.as_i64();
    const double eps = a.as_double(), alpha = a.as_double();
    const int b_min = a.as_int(), b_max = a.as_int(), linf = a.as_int();
    if (!a.ok) return nullptr;
    Py_buffer view;
    if (PyObject_GetBuffer(array, &view, PyBUF_C_CONTIGUOUS) != 0) return nullptr;
    if (view.ndim != 2 || view.itemsize != 4 || view.shape[0] > INT32_MAX || view.shape[1] > INT32_MAX) {
        PyBuffer_Release(&view);
        PyErr_SetString(PyExc_ValueError, "norms must be [M][n_seg]");
        return nullptr;
    }
    int b = 0, status;
    double gbar = 0.0;
    const auto* norms = static_cast<const float*>(view.buf);
    const int M = static_cast<int>(view.shape[0]), n_seg = static_cast<int>(view.shape[1]);
    Py_BEGIN_ALLOW_THREADS;
    status = linf ? a.lib->dq_select_bits_linf(norms, M, n_seg, t, T, eps, alpha, b_min, b_max, &b, &gbar)
                  : a.lib->dq_select_bits(norms, M, n_seg, t, T, eps, alpha, b_min, b_max, &b, &gbar);
    Py_END_ALLOW_THREADS;
    PyBuffer_Release(&view);
    return Py_BuildValue("iid", status, b, gbar);
}

// (plan, b) -> bytes
PyObject* py_packed_bytes(PyObject* module, args_t args, Py_ssize_t n)
{
    taker a(module, args, n, 2);
    const auto* plan = static_cast<const dq_plan_t*>(a.address());
    const int b = a.as_int();
    if (!a.ok) return nullptr;
    return PyLong_FromLongLong(a.lib->dq_packed_bytes(plan, b));
}

// ({name: address} of `functions`): the library that the other calls go to.
PyObject* py_bind(PyObject* module, PyObject* addresses)
{
    state* lib = state_of(module);
    if (!PyDict_Check(addresses)) {
        PyErr_SetString(PyExc_TypeError, "a dict of addresses");
        return nullptr;
    }
    lib->bound = false;
    const auto take = [&](const char* name) -> void* {
        PyObject* at = PyDict_GetItemString(addresses, name); // borrowed
        void* fn = at ? PyLong_AsVoidPtr(at) : nullptr;
        if (!fn && !PyErr_Occurred()) PyErr_Format(PyExc_ImportError, "%s: not in this library", name);
        return fn;
    };
#define X(fn)                                               \
    lib->fn = reinterpret_cast<decltype(&::fn)>(take(#fn)); \
    if (!lib->fn) return nullptr;
    DQ_FUNCTIONS(X)
#undef X
    lib->bound = true;
    Py_RETURN_NONE;
}

#define DQ_METHOD(name, fn) { name, reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(fn)), METH_FASTCALL, nullptr }
PyMethodDef methods[] = {
    { "bind", py_bind, METH_O, nullptr },
    DQ_METHOD("norm", py_norm),
    DQ_METHOD("quantize_pack", py_quantize_pack),
    DQ_METHOD("quantize_pack_v", py_quantize_pack_v),
    DQ_METHOD("norm_quantize_pack", py_norm_quantize_pack),
    DQ_METHOD("norm_bracket", py_norm_bracket),
    DQ_METHOD("bracketed", py_bracketed),
    DQ_METHOD("reduce", py_reduce),
    DQ_METHOD("reduce_update", py_reduce_update),
    DQ_METHOD("reduce_v", py_reduce_v),
    DQ_METHOD("reduce_update_v", py_reduce_update_v),
    DQ_METHOD("sign_pack", py_sign_pack),
    DQ_METHOD("sign_reduce", py_sign_reduce),
    DQ_METHOD("select_bits", py_select_bits),
    DQ_METHOD("packed_bytes", py_packed_bytes),
    { nullptr, nullptr, 0, nullptr },
};

template <typename T>
T same(T value)
{
    return value;
}
uint64_t number(void* address) { return reinterpret_cast<uint64_t>(address); }

// ctypes.PYFUNCTYPE(result, argument)(fn); nullptr, with an exception set, if that fails or one is set already
template <typename F>
PyObject* returning(PyObject* ctypes, const char* result, const char* argument, F* fn)
{
    if (PyErr_Occurred()) return nullptr;
    PyObject* result_type = PyObject_GetAttrString(ctypes, result);
    PyObject* argument_type = result_type ? PyObject_GetAttrString(ctypes, argument) : nullptr;
    PyObject* type = argument_type ? PyObject_CallMethod(ctypes, "PYFUNCTYPE", "OO", result_type, argument_type) : nullptr;
    PyObject* made = type ? PyObject_CallFunction(type, "K", static_cast<unsigned long long>(reinterpret_cast<uintptr_t>(fn))) : nullptr;
    Py_XDECREF(type);
    Py_XDECREF(argument_type);
    Py_XDECREF(result_type);
    return made;
}

int fill(PyObject* module)
{
    state* lib = state_of(module);
    PyObject* ctypes = PyImport_ImportModule("ctypes");
    if (!ctypes) return -1;
    lib->convert[INT32] = returning(ctypes, "c_int32", "c_int32", &same<int32_t>);
    lib->convert[UINT32] = returning(ctypes, "c_uint32", "c_uint32", &same<uint32_t>);
    lib->convert[INT64] = returning(ctypes, "c_int64", "c_int64", &same<int64_t>);
    lib->convert[UINT64] = returning(ctypes, "c_uint64", "c_uint64", &same<uint64_t>);
    lib->convert[ADDRESS] = returning(ctypes, "c_uint64", "c_void_p", &number);
    lib->convert[FLOAT32] = returning(ctypes, "c_float", "c_float", &same<float>);
    lib->convert[FLOAT64] = returning(ctypes, "c_double", "c_double", &same<double>);
    Py_DECREF(ctypes);
    for (const PyObject* convert : lib->convert)
        if (!convert) return -1;
    lib->data_ptr = PyUnicode_InternFromString("data_ptr");
    lib->stride = PyUnicode_InternFromString("stride");
    lib->size = PyUnicode_InternFromString("size");
    lib->shape = PyUnicode_InternFromString("shape");
    lib->zero = PyLong_FromLong(0);
    if (!lib->data_ptr || !lib->stride || !lib->size || !lib->shape || !lib->zero) return -1;
    static const char* const functions[] = {
#define X(fn) #fn,
        DQ_FUNCTIONS(X)
#undef X
    };
    PyObject* names = PyList_New(0);
    if (!names) return -1;
    for (const char* function : functions) {
        PyObject* name = PyUnicode_FromString(function);
        const bool added = name && PyList_Append(names, name) == 0;
        Py_XDECREF(name);
        if (!added) {
            Py_DECREF(names);
            return -1;
        }
    }
    if (PyModule_AddObject(module, "functions", names) != 0) {
        Py_DECREF(names);
        return -1;
    }
    return 0;
}

int visit_state(PyObject* module, visitproc visit, void* arg)
{
    if (state* lib = state_of(module))
        for (PyObject* convert : lib->convert) Py_VISIT(convert);
    return 0;
}
int clear_state(PyObject* module)
{
    if (state* lib = state_of(module)) {
        for (PyObject*& convert : lib->convert) Py_CLEAR(convert);
        Py_CLEAR(lib->data_ptr);
        Py_CLEAR(lib->stride);
        Py_CLEAR(lib->size);
        Py_CLEAR(lib->shape);
        Py_CLEAR(lib->zero);
        lib->bound = false;
    }
    return 0;
}
void free_state(void* module) { clear_state(static_cast<PyObject*>(module)); }

PyModuleDef_Slot slots[] = { { Py_mod_exec, reinterpret_cast<void*>(fill) }, { 0, nullptr } };
PyModuleDef definition = { PyModuleDef_HEAD_INIT, "_dqcall", "Calls of libdq.so's per-iteration entry points.", sizeof(state), methods, slots, visit_state, clear_state, free_state };

} // namespace

PyMODINIT_FUNC PyInit__dqcall(void) { return PyModuleDef_Init(&definition); }
