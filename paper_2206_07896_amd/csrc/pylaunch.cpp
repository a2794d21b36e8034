// pylaunch.cpp -- the marshalling of one launch from Python, without ctypes:
// parameters are packed into an array on the stack (the paper's parameter
// packing, Section III-C2) and spmd_launch is called with pointers to them.
//
// A launch costs the host 5 us through here (torch's stream lookup and the
// runtime's own launch included); building the same array out of ctypes
// objects took 14.5, twice what a reduction of 2^20 elements runs for.
//
// Only the plain forms of the arguments are taken (exact ints, tuples and
// lists; tensors by data_ptr()).  launch() returns None for anything else, a
// wrong argument count included, and the caller marshals or refuses it the
// general way.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>
#include <string.h>

#include "spmd.h"

namespace {

typedef int (*launch_fn)(int, spmd_dim3, spmd_dim3, size_t, void**, void*);
typedef const char* (*signature_fn)(int);
launch_fn g_launch = nullptr;
signature_fn g_signature = nullptr;
PyObject* g_data_ptr = nullptr;  // "data_ptr"

constexpr size_t MAX_ARGS = 16;

bool u32_of(PyObject* o, uint32_t* v) {
    if (!PyLong_CheckExact(o)) return false;
    *v = (uint32_t)PyLong_AsUnsignedLongLongMask(o);
    return true;
}

// An int, or a tuple of one to three.
bool dim_of(PyObject* o, spmd_dim3* d) {
    *d = {1, 1, 1};
    if (PyLong_CheckExact(o)) return u32_of(o, &d->x);
    if (!PyTuple_CheckExact(o)) return false;
    const Py_ssize_t n = PyTuple_GET_SIZE(o);
    if (n < 1 || n > 3) return false;
    uint32_t* f[3] = {&d->x, &d->y, &d->z};
    for (Py_ssize_t i = 0; i < n; ++i)
        if (!u32_of(PyTuple_GET_ITEM(o, i), f[i])) return false;
    return true;
}

// bind(address of spmd_launch, address of spmd_kernel_signature)
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 2) {
        PyErr_SetString(PyExc_TypeError, "bind(launch, signature)");
        return nullptr;
    }
    void* p[2];
    for (int i = 0; i < 2; ++i) {
        p[i] = PyLong_AsVoidPtr(a[i]);
        if (!p[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null function");
            return nullptr;
        }
    }
    g_launch = reinterpret_cast<launch_fn>(p[0]);
    g_signature = reinterpret_cast<signature_fn>(p[1]);
    Py_RETURN_NONE;
}

// launch(kernel, grid, block, dyn_shmem, args, stream) -> status, or None
PyObject* launch(PyObject*, PyObject* const* a, Py_ssize_t n) {
    spmd_dim3 grid, block;
    if (n != 6 || !g_launch || !PyLong_CheckExact(a[0]) || !PyLong_CheckExact(a[3]) || !PyLong_CheckExact(a[5]) ||
        !dim_of(a[1], &grid) || !dim_of(a[2], &block) || !(PyList_CheckExact(a[4]) || PyTuple_CheckExact(a[4])))
        Py_RETURN_NONE;
    const long kernel = PyLong_AsLong(a[0]);
    if (kernel < 0 || kernel > SPMD_NUM_KERNELS) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    const size_t shmem = (size_t)PyLong_AsUnsignedLongLongMask(a[3]);
    void* stream = reinterpret_cast<void*>((uintptr_t)PyLong_AsUnsignedLongLongMask(a[5]));
    const char* sig = g_signature((int)kernel);
    const Py_ssize_t nargs = PySequence_Fast_GET_SIZE(a[4]);
    if (!sig || strlen(sig) != (size_t)nargs || (size_t)nargs > MAX_ARGS) Py_RETURN_NONE;
    uint64_t value[MAX_ARGS];  // a uint32_t parameter is the low half (little-endian)
    void* args[MAX_ARGS];
    // the sequence may change under data_ptr(): hold each item over its call,
    // and look at the length again
    for (Py_ssize_t i = 0; i < nargs; ++i) {
        if (i >= PySequence_Fast_GET_SIZE(a[4])) Py_RETURN_NONE;
        PyObject* o = PySequence_Fast_GET_ITEM(a[4], i);
        args[i] = &value[i];
        if (PyLong_CheckExact(o)) {
            value[i] = PyLong_AsUnsignedLongLongMask(o);
        } else if (sig[i] != 'p' || PyLong_Check(o)) {
            Py_RETURN_NONE;
        } else if (o == Py_None) {
            value[i] = 0;
        } else {
            Py_INCREF(o);
            PyObject* p = PyObject_CallMethodNoArgs(o, g_data_ptr);
            Py_DECREF(o);
            if (!p) return nullptr;
            const bool whole = PyLong_CheckExact(p);
            if (whole) value[i] = PyLong_AsUnsignedLongLongMask(p);
            Py_DECREF(p);
            if (!whole) Py_RETURN_NONE;
        }
    }
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = g_launch((int)kernel, grid, block, shmem, args, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

PyMethodDef methods[] = {
    {"bind", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(bind)), METH_FASTCALL, nullptr},
    {"launch", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(launch)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_launch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__launch(void) {
    g_data_ptr = PyUnicode_InternFromString("data_ptr");
    return g_data_ptr ? PyModule_Create(&module) : nullptr;
}
