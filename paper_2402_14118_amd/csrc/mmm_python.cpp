// CPython entry points for the three calls a program makes per step (mmm_build_maps, mmm_matmul,
// mmm_matmul_fused).  They do what the ctypes functions of binding.py do -- marshal integers and call
// the C ABI -- at 0.3 instead of about 3 us per call: a small problem is bound by the host, where a
// kernel launch alone takes 3.5 us.  Pointers are passed as integers (None = NULL).  The GIL is
// released around the call, as ctypes does.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include "mmm.h"

namespace {

// integer arguments; reading stops at the first bad one
struct Args {
    PyObject *const *v;
    bool ok = true;
    void *ptr(int i)
    {
        if (!ok || v[i] == Py_None) return nullptr;
        void *p = PyLong_AsVoidPtr(v[i]);
        if (p == nullptr && PyErr_Occurred()) ok = false;
        return p;
    }
    int64_t num(int i)
    {
        if (!ok) return 0;
        const long long n = PyLong_AsLongLong(v[i]);
        if (n == -1 && PyErr_Occurred()) ok = false;
        return (int64_t)n;
    }
    float real(int i)
    {
        if (!ok) return 0.f;
        const double d = PyFloat_AsDouble(v[i]);
        if (d == -1.0 && PyErr_Occurred()) ok = false;
        return (float)d;
    }
};

bool arity(const char *name, Py_ssize_t n, Py_ssize_t want)
{
    if (n == want) return true;
    PyErr_Format(PyExc_TypeError, "%s takes %zd arguments, got %zd", name, want, n);
    return false;
}

// build_maps(maps, dtype, X, ldx, has_ma, pred, threshold, keep_a, Y, ldy, has_mb, block_width, keep_rows, keep_blocks, stream)
PyObject *build_maps(PyObject *, PyObject *const *v, Py_ssize_t n)
{
    if (!arity("build_maps", n, 15)) return nullptr;
    Args a{v};
    mmm_maps *maps = static_cast<mmm_maps *>(a.ptr(0));
    const mmm_dtype dt = (mmm_dtype)a.num(1);
    const void *X = a.ptr(2);
    const int64_t ldx = a.num(3);
    const bool has_ma = a.num(4) != 0;
    const mmm_mask_a ma{(int32_t)a.num(5), a.real(6), static_cast<const uint64_t *>(a.ptr(7))};
    const void *Y = a.ptr(8);
    const int64_t ldy = a.num(9);
    const bool has_mb = a.num(10) != 0;
    const mmm_mask_b mb{(int32_t)a.num(11), static_cast<const uint64_t *>(a.ptr(12)), static_cast<const uint64_t *>(a.ptr(13))};
    void *stream = a.ptr(14);
    if (!a.ok) return nullptr;
    mmm_status st;
    Py_BEGIN_ALLOW_THREADS
    st = mmm_build_maps(maps, dt, X, ldx, has_ma ? &ma : nullptr, Y, ldy, has_mb ? &mb : nullptr, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
}

// matmul(maps, dtype, X, ldx, Y, ldy, C, ldc, accumulate, stream)
PyObject *matmul(PyObject *, PyObject *const *v, Py_ssize_t n)
{
    if (!arity("matmul", n, 10)) return nullptr;
    Args a{v};
    const mmm_maps *maps = static_cast<const mmm_maps *>(a.ptr(0));
    const mmm_dtype dt = (mmm_dtype)a.num(1);
    const void *X = a.ptr(2);
    const int64_t ldx = a.num(3);
    const void *Y = a.ptr(4);
    const int64_t ldy = a.num(5);
    void *C = a.ptr(6);
    const int64_t ldc = a.num(7);
    const int32_t acc = (int32_t)a.num(8);
    void *stream = a.ptr(9);
    if (!a.ok) return nullptr;
    mmm_status st;
    Py_BEGIN_ALLOW_THREADS
    st = mmm_matmul(maps, dt, X, ldx, Y, ldy, C, ldc, acc, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
}

// matmul_fused(maps, dtype, X, ldx, pred, threshold, keep_a, Y, ldy, C, ldc, accumulate, stream)
PyObject *matmul_fused(PyObject *, PyObject *const *v, Py_ssize_t n)
{
    if (!arity("matmul_fused", n, 13)) return nullptr;
    Args a{v};
    const mmm_maps *maps = static_cast<const mmm_maps *>(a.ptr(0));
    const mmm_dtype dt = (mmm_dtype)a.num(1);
    const void *X = a.ptr(2);
    const int64_t ldx = a.num(3);
    const mmm_mask_a ma{(int32_t)a.num(4), a.real(5), static_cast<const uint64_t *>(a.ptr(6))};
    const void *Y = a.ptr(7);
    const int64_t ldy = a.num(8);
    void *C = a.ptr(9);
    const int64_t ldc = a.num(10);
    const int32_t acc = (int32_t)a.num(11);
    void *stream = a.ptr(12);
    if (!a.ok) return nullptr;
    mmm_status st;
    Py_BEGIN_ALLOW_THREADS
    st = mmm_matmul_fused(maps, dt, X, ldx, &ma, Y, ldy, C, ldc, acc, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
}

PyMethodDef methods[] = {
    {"build_maps", (PyCFunction)(void (*)(void))build_maps, METH_FASTCALL, nullptr},
    {"matmul", (PyCFunction)(void (*)(void))matmul, METH_FASTCALL, nullptr},
    {"matmul_fused", (PyCFunction)(void (*)(void))matmul_fused, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_mmm_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}   // namespace

PyMODINIT_FUNC PyInit__mmm_native(void) { return PyModule_Create(&module); }
