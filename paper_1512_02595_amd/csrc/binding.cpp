// CPython module `_binding`: the per-call entry points of the CTC library without ctypes in between.
//
// A call through ctypes spends about 10 us on converting its arguments (three numpy arrays to pointers,
// a dozen integers to C objects), as long as a small minibatch takes on the GPU; here the arrays are taken
// by the buffer protocol and the integers by PyLong_As...: under 1 us.  The functions take positional
// arguments only, in the order of the C functions, and return the status; `bind` is given the
// addresses of the library's functions (ctc.py loads the library).  An array that is not a contiguous
// int32 buffer makes a call return None: ctc.py then converts it and calls again.
// The GIL is released around the library call, as ctypes does.

#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstdint>

#include "ctc_mi355x.h"

namespace {

using HostCall = ctc_status_t (*)(const void*, const int32_t*, const int32_t*, const int32_t*, int, int, int, int,
                                  ctc_dtype_t, float*, void*, void*, size_t, hipStream_t);
using BestCall = ctc_status_t (*)(const void*, const int32_t*, const int32_t*, const int32_t*, int, int, int, int,
                                  ctc_dtype_t, float*, int32_t*, void*, size_t, hipStream_t);
using DeviceCall = ctc_status_t (*)(const void*, const int32_t*, const int32_t*, const int32_t*, int, int, int, int, int,
                                    ctc_dtype_t, float*, void*, int32_t*, void*, size_t, hipStream_t);

HostCall g_loss_and_grad;
BestCall g_best_path;
DeviceCall g_loss_and_grad_device;

// None is the null pointer.
bool address(PyObject* o, void** out)
{
    *out = o == Py_None ? nullptr : PyLong_AsVoidPtr(o);
    return *out || !PyErr_Occurred();
}
bool integer(PyObject* o, int* out)
{
    long v = 0;
    if (PyLong_Check(o)) {
        v = PyLong_AsLong(o);
    } else {                                    // (numpy integers and their like)
        PyObject* index = PyNumber_Long(o);
        if (!index) return false;
        v = PyLong_AsLong(index);
        Py_DECREF(index);
    }
    if (v == -1 && PyErr_Occurred()) return false;
    *out = static_cast<int>(v);
    return true;
}

// A contiguous int32 buffer, held until the call has returned; None is a null pointer.
struct Ints {
    Py_buffer view{};
    bool held = false;
    const int32_t* data = nullptr;
    ~Ints()
    {
        if (held) PyBuffer_Release(&view);
    }
    bool take(PyObject* o)
    {
        if (o == Py_None) return true;
        if (!PyObject_CheckBuffer(o)) return false;
        if (PyObject_GetBuffer(o, &view, PyBUF_C_CONTIGUOUS | PyBUF_FORMAT) != 0) {
            PyErr_Clear();
            return false;
        }
        held = true;
        const char* f = view.format;
        if (view.itemsize != 4 || !f || f[0] != 'i' || f[1] != 0) return false;
        data = static_cast<const int32_t*>(view.buf);
        return true;
    }
};

bool arity(Py_ssize_t n, Py_ssize_t want)
{
    if (n == want) return true;
    PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, n);
    return false;
}

// (activations, flat_labels, label_lengths, input_lengths, T, B, A, blank, dtype, costs, grads or alignment,
//  workspace, workspace_bytes, stream)
template <typename Call>
PyObject* host_call(Call call, PyObject* const* a, Py_ssize_t n)
{
    if (!arity(n, 14)) return nullptr;
    void *x, *costs, *out, *ws, *bytes, *stream;
    int T, B, A, blank, dtype;
    if (!address(a[0], &x) || !integer(a[4], &T) || !integer(a[5], &B) || !integer(a[6], &A) || !integer(a[7], &blank) ||
        !integer(a[8], &dtype) || !address(a[9], &costs) || !address(a[10], &out) || !address(a[11], &ws) ||
        !address(a[12], &bytes) || !address(a[13], &stream))
        return nullptr;
    Ints labels, label_lengths, input_lengths;
    if (!labels.take(a[1]) || !label_lengths.take(a[2]) || !input_lengths.take(a[3])) Py_RETURN_NONE;
    ctc_status_t st;
    Py_BEGIN_ALLOW_THREADS
    st = call(x, labels.data, label_lengths.data, input_lengths.data, T, B, A, blank, static_cast<ctc_dtype_t>(dtype),
              static_cast<float*>(costs), static_cast<int32_t*>(out), ws,
              reinterpret_cast<size_t>(bytes), static_cast<hipStream_t>(stream));
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
}

PyObject* loss_and_grad(PyObject*, PyObject* const* a, Py_ssize_t n) { return host_call(g_loss_and_grad, a, n); }
PyObject* best_path(PyObject*, PyObject* const* a, Py_ssize_t n) { return host_call(g_best_path, a, n); }

// (activations, labels, label_lengths, input_lengths, max_label_length, T, B, A, blank, dtype, costs, grads, status,
//  workspace, workspace_bytes, stream)
PyObject* loss_and_grad_device(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    if (!arity(n, 16)) return nullptr;
    void *x, *labels, *label_lengths, *input_lengths, *costs, *grads, *status, *ws, *bytes, *stream;
    int max_label, T, B, A, blank, dtype;
    if (!address(a[0], &x) || !address(a[1], &labels) || !address(a[2], &label_lengths) || !address(a[3], &input_lengths) ||
        !integer(a[4], &max_label) || !integer(a[5], &T) || !integer(a[6], &B) || !integer(a[7], &A) || !integer(a[8], &blank) ||
        !integer(a[9], &dtype) || !address(a[10], &costs) || !address(a[11], &grads) || !address(a[12], &status) ||
        !address(a[13], &ws) || !address(a[14], &bytes) || !address(a[15], &stream))
        return nullptr;
    ctc_status_t st;
    Py_BEGIN_ALLOW_THREADS
    st = g_loss_and_grad_device(x, static_cast<const int32_t*>(labels), static_cast<const int32_t*>(label_lengths),
                                static_cast<const int32_t*>(input_lengths), max_label, T, B, A, blank,
                                static_cast<ctc_dtype_t>(dtype), static_cast<float*>(costs), grads,
                                static_cast<int32_t*>(status), ws, reinterpret_cast<size_t>(bytes),
                                static_cast<hipStream_t>(stream));
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
}

PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    void *f, *g, *h;
    if (!arity(n, 3) || !address(a[0], &f) || !address(a[1], &g) || !address(a[2], &h)) return nullptr;
    g_loss_and_grad = reinterpret_cast<HostCall>(f);
    g_best_path = reinterpret_cast<BestCall>(g);
    g_loss_and_grad_device = reinterpret_cast<DeviceCall>(h);
    Py_RETURN_NONE;
}

PyMethodDef g_methods[] = {
    {"bind", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(bind)), METH_FASTCALL,
     "Addresses of ctc_loss_and_grad, ctc_best_path and ctc_loss_and_grad_device."},
    {"loss_and_grad", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(loss_and_grad)), METH_FASTCALL, nullptr},
    {"best_path", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(best_path)), METH_FASTCALL, nullptr},
    {"loss_and_grad_device", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(loss_and_grad_device)), METH_FASTCALL,
     nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void) { return PyModule_Create(&g_module); }
