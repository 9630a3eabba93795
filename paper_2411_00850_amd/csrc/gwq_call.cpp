// Python extension module _call: gwq.linear and gwq.linear_bf16 called the plain way - activations in, result allocated, current
// stream - without the interpreter in between.  The binding's own way through ctypes took 8.0 us of host time a call, half of it
// for attributes, the C struct and the marshalling of eight arguments, where the kernel of a 4096 x 4096 layer at one row
// takes 5: a token of a program that calls its projections this way is bound by it.  Here a call reads the layer's fields, which
// are looked at anew each time, and enqueues.
//
// Whatever is not the plain case - another argument, a tensor that the checks below do not know to be right - is handed back
// (None), and the binding goes its own way, which also words the errors.
#include <Python.h>

#include <ATen/ATen.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/object_ptr.h>

#include "gwq.h"

namespace {

typedef gwq_status (*LinearFn)(const gwq_packed *, const void *, int32_t, void *, void *, size_t, void *);
typedef gwq_status (*LayoutFn)(int32_t, int32_t, int32_t, int32_t, uint32_t, int32_t, gwq_sizes *);
LinearFn g_linear[2];                                   // FP16, bfloat16
LayoutFn g_layout;
PyObject *g_raw_stream, *g_current_device;              // torch._C functions: the stream's handle; the device
PyObject *g_scalar_names[6], *g_tensor_names[7];

// An integer attribute of `o`; false if it is none.
bool integer(PyObject *o, PyObject *name, int64_t low, int64_t high, int64_t &out)
{
    PyObject *v = PyObject_GetAttr(o, name);
    if (!v) return false;
    out = PyLong_Check(v) ? PyLong_AsLongLong(v) : -1;
    Py_DECREF(v);
    return out >= low && out <= high && !PyErr_Occurred();
}

// The layer's C struct; false where a field is not what the binding's own way would take.
bool read_layer(PyObject *layer, gwq_packed &P)
{
    int64_t s[6];
    constexpr int64_t kInt = 0x7FFFFFFF;
    for (int i = 0; i < 6; ++i)
        if (!integer(layer, g_scalar_names[i], 0, i == 5 ? (int64_t)1 << 40 : kInt, s[i])) return false;
    P.N = (int32_t)s[0]; P.K = (int32_t)s[1]; P.bits = (int32_t)s[2]; P.group = (int32_t)s[3];
    P.outlier_ppm = (uint32_t)s[4]; P.n_outliers = s[5];
    void *ptr[7];
    for (int i = 0; i < 7; ++i) {
        THPObjectPtr t(PyObject_GetAttr(layer, g_tensor_names[i]));   // (the layer keeps the tensor)
        if (!t.get()) return false;
        const bool none = i == 6 && t.get() == Py_None;
        if (!none && !THPVariable_CheckExact(t.get())) return false;
        ptr[i] = none ? nullptr : THPVariable_Unpack(t.get()).data_ptr();
    }
    P.qweight = static_cast<uint32_t *>(ptr[0]); P.scales = static_cast<uint16_t *>(ptr[1]); P.zeros = static_cast<uint8_t *>(ptr[2]);
    P.row_ptr = static_cast<int32_t *>(ptr[3]); P.col_idx = static_cast<uint16_t *>(ptr[4]); P.out_val = static_cast<uint16_t *>(ptr[5]);
    P.index = ptr[6];
    return true;
}

// The current stream of the current device, as an integer handle.
bool current_stream(void *&stream)
{
    THPObjectPtr device(PyObject_CallNoArgs(g_current_device));
    if (!device.get()) return false;
    THPObjectPtr handle(PyObject_CallOneArg(g_raw_stream, device.get()));
    if (!handle.get()) return false;
    stream = PyLong_AsVoidPtr(handle.get());
    return !PyErr_Occurred();
}

PyObject *not_plain()
{
    PyErr_Clear();
    Py_RETURN_NONE;
}

// call(layer, X, out or None, bf16) -> the result; (status, None) where the library refuses; None: not the plain case, nothing done.
PyObject *call(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != 4) { PyErr_SetString(PyExc_TypeError, "call(layer, X, out, bf16)"); return nullptr; }
    HANDLE_TH_ERRORS                                    // as torch words its own, running out of memory among them
    const int bf16 = args[3] == Py_True;
    const at::ScalarType type = bf16 ? at::kBFloat16 : at::kHalf;
    gwq_packed P;
    if (!THPVariable_CheckExact(args[1]) || !read_layer(args[0], P)) return not_plain();
    const at::Tensor &X = THPVariable_Unpack(args[1]);
    if (!X.is_cuda() || X.scalar_type() != type || X.dim() != 2 || !X.is_contiguous() || X.size(1) != P.K || X.size(0) > 0x7FFFFFFF) return not_plain();
    const int32_t M = (int32_t)X.size(0);
    at::Tensor Y, workspace;
    if (args[2] == Py_None) {
        Y = at::empty({M, P.N}, X.options());
    } else {
        if (!THPVariable_CheckExact(args[2])) return not_plain();
        Y = THPVariable_Unpack(args[2]);
        if (!Y.is_cuda() || Y.scalar_type() != type || Y.dim() != 2 || !Y.is_contiguous() || Y.size(0) != M || Y.size(1) != P.N) return not_plain();
    }
    size_t bytes = 0;
    if (M > 16) {                                   // as the binding's _workspace_bytes: the scratch, and a copy of X where it does not fit there
        gwq_sizes sz;
        if (g_layout(P.N, P.K, P.bits, P.group, P.outlier_ppm, M, &sz) != GWQ_OK) return not_plain();
        const size_t copy = ((size_t)M + 15) / 16 * 16 * (size_t)P.K * 2;
        bytes = sz.linear_workspace + (2 * copy > sz.linear_scratch ? copy : 0);
        workspace = at::empty({(int64_t)bytes}, X.options().dtype(at::kByte));
    }
    void *stream;
    if (!current_stream(stream)) return nullptr;
    const void *x = X.data_ptr();
    void *y = Y.data_ptr(), *w = bytes ? workspace.data_ptr() : nullptr;
    gwq_status status;
    Py_BEGIN_ALLOW_THREADS
    status = g_linear[bf16](&P, x, M, y, w, bytes, stream);
    Py_END_ALLOW_THREADS
    if (status != GWQ_OK) return Py_BuildValue("(iO)", (int)status, Py_None);
    if (args[2] != Py_None) { Py_INCREF(args[2]); return args[2]; }
    return THPVariable_Wrap(std::move(Y));
    END_HANDLE_TH_ERRORS
}

// bind(address of gwq_linear, of gwq_linear_bf16, of gwq_layout, raw stream function, current device function)
PyObject *bind(PyObject *, PyObject *args)
{
    unsigned long long a, b, c;
    PyObject *stream, *device;
    if (!PyArg_ParseTuple(args, "KKKOO", &a, &b, &c, &stream, &device)) return nullptr;
    g_linear[0] = reinterpret_cast<LinearFn>(a);
    g_linear[1] = reinterpret_cast<LinearFn>(b);
    g_layout = reinterpret_cast<LayoutFn>(c);
    Py_INCREF(stream); Py_INCREF(device);
    g_raw_stream = stream; g_current_device = device;
    Py_RETURN_NONE;
}

PyMethodDef g_methods[] = {{"call", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(call)), METH_FASTCALL, nullptr},
                           {"bind", bind, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_call", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__call()
{
    const char *scalars[6] = {"N", "K", "bits", "group", "ppm", "n_outliers"};
    const char *tensors[7] = {"qweight", "scales", "zeros", "row_ptr", "col_idx", "out_val", "index"};
    for (int i = 0; i < 6; ++i)
        if (!(g_scalar_names[i] = PyUnicode_InternFromString(scalars[i]))) return nullptr;
    for (int i = 0; i < 7; ++i)
        if (!(g_tensor_names[i] = PyUnicode_InternFromString(tensors[i]))) return nullptr;
    PyObject *m = PyModule_Create(&g_module);
    if (m && PyModule_AddStringConstant(m, "built_for", GWQ_BUILT_FOR) < 0) Py_CLEAR(m);
    return m;
}
