// Argument marshalling of the short calls (module _marshal): append, verdict and conditional verdict take their tensors as they are,
// check them and call the library.  A launch takes about 4 us of host time; the checks and conversions of up to eight tensors took
// 2 to 3 more in Python, on calls whose kernels take 3 to 6.
//
// Every function returns the library's status, or kOther when an argument is not the plain one it is made for (another type, dtype or
// device, not contiguous, a size that does not match, a tensor subclass or mode): the caller then goes its general way, which words
// the error.  Nothing is decided here that the general way would decide otherwise.
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>

#include "atts.h"

namespace {

constexpr long kOther = 1;                       // statuses are <= 0
PyObject* g_device = nullptr;                    // torch._C._cuda_getDevice, torch._C._cuda_getCurrentRawStream
PyObject* g_stream = nullptr;

struct Array {
    void* data = nullptr;
    int64_t n = 0;
};

// a contiguous device tensor of the type, or (optional) None
bool take(PyObject* o, at::ScalarType type, bool optional, Array& out) {
    if (o == Py_None) return optional;
    if (!THPVariable_CheckExact(o)) return false;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_cuda() || t.scalar_type() != type || !t.is_contiguous()) return false;
    out.data = t.data_ptr();
    out.n = t.numel();
    return true;
}

bool take_handle(PyObject* o, void*& out) {
    if (!PyLong_CheckExact(o)) return false;
    out = PyLong_AsVoidPtr(o);
    return out != nullptr && !PyErr_Occurred();
}

// exact floats only (anything else is converted by the general way)
bool take_levels(PyObject* o, double (&out)[ATTS_MAX_ALPHAS], int32_t& n) {
    const bool list = PyList_CheckExact(o), tuple = PyTuple_CheckExact(o);
    if (!list && !tuple) return false;
    const Py_ssize_t len = list ? PyList_GET_SIZE(o) : PyTuple_GET_SIZE(o);
    if (len < 1 || len > ATTS_MAX_ALPHAS) return false;
    for (Py_ssize_t i = 0; i < len; ++i) {
        PyObject* x = list ? PyList_GET_ITEM(o, i) : PyTuple_GET_ITEM(o, i);
        if (!PyFloat_CheckExact(x)) return false;
        out[i] = PyFloat_AS_DOUBLE(x);
    }
    n = (int32_t)len;
    return true;
}

// the current stream of the current device
bool take_stream(void*& out) {
    PyObject* device = PyObject_CallNoArgs(g_device);
    if (!device) return false;
    PyObject* stream = PyObject_CallOneArg(g_stream, device);
    Py_DECREF(device);
    if (!stream) return false;
    out = PyLong_AsVoidPtr(stream);
    Py_DECREF(stream);
    return !PyErr_Occurred();
}

template <typename F>
PyObject* guarded(F&& call) {
    long status = kOther;
    try {
        if (g_stream && !at::impl::torch_function_mode_enabled()) status = call();
    } catch (...) {                              // a tensor without storage, and the like
        status = kOther;
    }
    PyErr_Clear();
    return PyLong_FromLong(status);
}

PyObject* setup(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 2) {
        PyErr_SetString(PyExc_TypeError, "setup(current_device, current_raw_stream)");
        return nullptr;
    }
    Py_INCREF(a[0]);
    Py_INCREF(a[1]);
    Py_XSETREF(g_device, a[0]);
    Py_XSETREF(g_stream, a[1]);
    Py_RETURN_NONE;
}

PyObject* calibrate_online(PyObject*, PyObject* const* a, Py_ssize_t n) {       // handle, new_scores
    return guarded([&]() -> long {
        void *handle, *stream;
        Array scores;
        if (n != 2 || !take_handle(a[0], handle) || !take(a[1], at::kFloat, false, scores) || !take_stream(stream)) return kOther;
        int32_t rc;
        Py_BEGIN_ALLOW_THREADS
        rc = atts_calibrate_online(static_cast<atts_calib*>(handle), static_cast<const float*>(scores.data), scores.n, stream);
        Py_END_ALLOW_THREADS
        return rc;
    });
}

PyObject* classify_ordinal(PyObject*, PyObject* const* a, Py_ssize_t n) {       // handle, test, alphas, ranks, pvalues, classes, thresholds
    return guarded([&]() -> long {
        void *handle, *stream;
        Array test, ranks, pvalues, classes, thresholds;
        double alphas[ATTS_MAX_ALPHAS];
        int32_t n_alpha;
        if (n != 7 || !take_handle(a[0], handle) || !take(a[1], at::kFloat, false, test) || !take_levels(a[2], alphas, n_alpha) ||
            !take(a[3], at::kInt, true, ranks) || !take(a[4], at::kFloat, true, pvalues) || !take(a[5], at::kByte, false, classes) ||
            !take(a[6], at::kFloat, true, thresholds))
            return kOther;
        if ((a[3] != Py_None && ranks.n != test.n) || (a[4] != Py_None && pvalues.n != test.n) || classes.n != test.n ||
            (a[6] != Py_None && thresholds.n != n_alpha) || !take_stream(stream))
            return kOther;
        int32_t rc;
        Py_BEGIN_ALLOW_THREADS
        rc = atts_classify_ordinal(static_cast<const atts_calib*>(handle), static_cast<const float*>(test.data), test.n, alphas, n_alpha,
                                   static_cast<int32_t*>(ranks.data), static_cast<float*>(pvalues.data),
                                   static_cast<uint8_t*>(classes.data), static_cast<float*>(thresholds.data), stream);
        Py_END_ALLOW_THREADS
        return rc;
    });
}

PyObject* classify_conditional(PyObject*, PyObject* const* a, Py_ssize_t n) {   // cal, cal_off, test, test_off, alphas, ranks, pvalues, classes
    return guarded([&]() -> long {
        void* stream;
        Array cal, cal_off, test, test_off, ranks, pvalues, classes;
        double alphas[ATTS_MAX_ALPHAS];
        int32_t n_alpha;
        if (n != 8 || !take(a[0], at::kFloat, false, cal) || !take(a[1], at::kLong, false, cal_off) || !take(a[2], at::kFloat, false, test) ||
            !take(a[3], at::kLong, false, test_off) || !take_levels(a[4], alphas, n_alpha) || !take(a[5], at::kInt, false, ranks) ||
            !take(a[6], at::kFloat, true, pvalues) || !take(a[7], at::kByte, false, classes))
            return kOther;
        // empty arrays (no address) and mismatches go the general way
        if (cal_off.n < 1 || test_off.n != cal_off.n || cal.n == 0 || test.n == 0 || ranks.n != test.n || classes.n != test.n ||
            (a[6] != Py_None && pvalues.n != test.n) || !take_stream(stream))
            return kOther;
        int32_t rc;
        Py_BEGIN_ALLOW_THREADS
        rc = atts_classify_conditional(static_cast<const float*>(cal.data), static_cast<const int64_t*>(cal_off.data),
                                       static_cast<const float*>(test.data), static_cast<const int64_t*>(test_off.data), cal_off.n - 1, alphas,
                                       n_alpha, static_cast<int32_t*>(ranks.data), static_cast<float*>(pvalues.data),
                                       static_cast<uint8_t*>(classes.data), stream);
        Py_END_ALLOW_THREADS
        return rc;
    });
}

#define ATTS_METHOD(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {ATTS_METHOD(setup), ATTS_METHOD(calibrate_online), ATTS_METHOD(classify_ordinal), ATTS_METHOD(classify_conditional),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() {
    PyObject* m = PyModule_Create(&module);
    if (m) PyModule_AddIntConstant(m, "OTHER", kOther);
    return m;
}
