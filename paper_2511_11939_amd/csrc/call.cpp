// The way from Python into the library for the usual call: pointers of three tensors, whole numbers,
// the current stream.  Bound by the host: a product of 256 x 256 matrices takes the GPU 3.4 us, and a call through
// ctypes with its arguments looked after in Python took 5.2.  Anything unusual (raw pointers, other kinds of
// numbers, sizes out of range) is declined with None and takes the Python way, so what is
// accepted and what is raised stays where it was.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstdint>

#include "../../include/prism_gemm.h"
#include "../../include/prism_scan.h"

namespace {

decltype(&prism_gemm) g_gemm = nullptr;
decltype(&prism_gemm_batched) g_gemm_batched = nullptr;
decltype(&prism_scan_u32) g_scan = nullptr;
PyObject *g_data_ptr = nullptr, *g_numel = nullptr, *g_element_size = nullptr;  // names
PyObject *g_device = nullptr, *g_raw_stream = nullptr;                          // the current device, a device's current stream
PyTypeObject* g_desc_type = nullptr;

// false: not a whole number of 64 bits (no error is left behind)
bool whole(PyObject* o, int64_t* out)
{
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    *out = PyLong_AsLongLongAndOverflow(o, &overflow);
    return overflow == 0;
}
bool method_whole(PyObject* tensor, PyObject* name, int64_t* out)
{
    PyObject* r = PyObject_CallMethodNoArgs(tensor, name);
    if (!r) {
        PyErr_Clear();
        return false;
    }
    const bool ok = whole(r, out);
    Py_DECREF(r);
    return ok;
}
bool pointer(PyObject* o, void** out)
{
    int64_t v = 0;
    if (!method_whole(o, g_data_ptr, &v)) return false;
    *out = reinterpret_cast<void*>(static_cast<uintptr_t>(v));
    return true;
}
bool current_stream(void** out)
{
    PyObject* device = PyObject_CallNoArgs(g_device);
    PyObject* stream = device ? PyObject_CallOneArg(g_raw_stream, device) : nullptr;
    Py_XDECREF(device);
    if (!stream) {
        PyErr_Clear();
        return false;
    }
    int64_t v = 0;
    const bool ok = whole(stream, &v);
    Py_DECREF(stream);
    *out = reinterpret_cast<void*>(static_cast<uintptr_t>(v));
    return ok;
}

// bind(gemm, gemm_batched, scan, GemmDesc, device, raw_stream): addresses of the library's entry points, the descriptor's
// type, and torch's functions for the current device and its raw stream
PyObject* bind(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    int64_t f[3];
    if (n != 6 || !whole(args[0], &f[0]) || !whole(args[1], &f[1]) || !whole(args[2], &f[2]) || !PyType_Check(args[3])) {
        PyErr_SetString(PyExc_TypeError, "bind: three addresses, a type, two functions");
        return nullptr;
    }
    g_gemm = reinterpret_cast<decltype(g_gemm)>(static_cast<uintptr_t>(f[0]));
    g_gemm_batched = reinterpret_cast<decltype(g_gemm_batched)>(static_cast<uintptr_t>(f[1]));
    g_scan = reinterpret_cast<decltype(g_scan)>(static_cast<uintptr_t>(f[2]));
    for (int i = 3; i < 6; ++i) Py_INCREF(args[i]);  // (kept for good: bound once per library)
    g_desc_type = reinterpret_cast<PyTypeObject*>(args[3]);
    g_device = args[4];
    g_raw_stream = args[5];
    Py_RETURN_NONE;
}

// gemm(A, B, C, M, N, K, desc, lda, ldb, ldc, batch, strideA, strideB, strideC) on the current stream -> status, or None
PyObject* gemm(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    void *a, *b, *c, *stream;
    int64_t M, N, K, batch;
    if (n != 14 || !g_gemm || Py_TYPE(args[6]) != g_desc_type || !whole(args[3], &M) || !whole(args[4], &N) || !whole(args[5], &K) ||
        !whole(args[10], &batch) || !pointer(args[0], &a) || !pointer(args[1], &b) || !pointer(args[2], &c) || !current_stream(&stream))
        Py_RETURN_NONE;
    Py_buffer view;
    if (PyObject_GetBuffer(args[6], &view, PyBUF_SIMPLE) != 0) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    const auto* desc = static_cast<const prism_gemm_desc_t*>(view.buf);
    const int64_t packed[3] = {desc->layout_a == PRISM_ROW_MAJOR ? K : M, desc->layout_b == PRISM_ROW_MAJOR ? N : K, desc->layout_c == PRISM_ROW_MAJOR ? N : M};
    int64_t ld[3], stride[3];
    bool ok = view.len == static_cast<Py_ssize_t>(sizeof(prism_gemm_desc_t)), strides = false;
    // (products of sizes beyond 2^31 are left to Python's whole numbers)
    ok = ok && M < (int64_t{1} << 31) && N < (int64_t{1} << 31) && K < (int64_t{1} << 31) && M >= 0 && N >= 0 && K >= 0;
    const int64_t spans[3] = {ok ? M * K : 0, ok ? K * N : 0, ok ? M * N : 0};
    for (int i = 0; i < 3 && ok; ++i) {
        if (args[7 + i] == Py_None) ld[i] = packed[i];
        else ok = whole(args[7 + i], &ld[i]);
        if (args[11 + i] == Py_None) stride[i] = spans[i];
        else ok = ok && whole(args[11 + i], &stride[i]), strides = true;
        if (ok && ld[i] < 1) ld[i] = 1;
    }
    long status = 0;
    if (ok) {
        Py_BEGIN_ALLOW_THREADS
        if (batch == 1 && !strides) status = g_gemm(desc, M, N, K, a, ld[0], b, ld[1], c, ld[2], stream);
        else status = g_gemm_batched(desc, M, N, K, a, ld[0], stride[0], b, ld[1], stride[1], c, ld[2], stride[2], batch, stream);
        Py_END_ALLOW_THREADS
    }
    PyBuffer_Release(&view);
    if (!ok) Py_RETURN_NONE;
    return PyLong_FromLong(status);
}

// scan(input, output, n, workspace) on the current stream -> status, or None
PyObject* scan(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    void *in, *out, *workspace, *stream;
    int64_t count, numel, size;
    if (n != 4 || !g_scan || !whole(args[2], &count) || !pointer(args[0], &in) || !pointer(args[1], &out) || !pointer(args[3], &workspace) ||
        !method_whole(args[3], g_numel, &numel) || !method_whole(args[3], g_element_size, &size) || !current_stream(&stream))
        Py_RETURN_NONE;
    long status;
    Py_BEGIN_ALLOW_THREADS
    status = g_scan(static_cast<const uint32_t*>(in), static_cast<uint32_t*>(out), count, workspace, static_cast<size_t>(numel * size), stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

PyMethodDef g_methods[] = {
    {"bind", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(bind)), METH_FASTCALL, nullptr},
    {"gemm", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(gemm)), METH_FASTCALL, nullptr},
    {"scan", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(scan)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_call", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__call(void)
{
    g_data_ptr = PyUnicode_InternFromString("data_ptr");
    g_numel = PyUnicode_InternFromString("numel");
    g_element_size = PyUnicode_InternFromString("element_size");
    if (!g_data_ptr || !g_numel || !g_element_size) return nullptr;
    return PyModule_Create(&g_module);
}
