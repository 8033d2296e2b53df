// The run-time calls of binding.py, marshalled natively: tensors in, the C ABI's status out.
//
// A small layer's kernel takes 3 - 5 us.  Marshalling a call in Python -- an attribute check and a pointer object per
// tensor, the current stream, the conversions of a ctypes call -- took 5.5 us beside it, so a program that launches such
// layers one after another waited for its own host thread: 56x56x64 -> 64 3x3 for one image 10.5 us a call.  Here the checks
// are the same ones on the tensor objects themselves, about 0.4 us a call.
//
// Nothing is kept from one call for the next, and nothing is allocated.  The interpreter lock is released around the library
// call (a launch may wait for the device's queue).
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <c10/core/impl/DeviceGuardImplInterface.h>
#include <torch/csrc/DynamicTypes.h>
#include <torch/csrc/autograd/python_variable.h>

#include "deepgemm_hip.h"

namespace {

PyObject *g_raw_stream = nullptr;        // torch._C._cuda_getCurrentRawStream
PyObject *g_stream_attr = nullptr;       // "cuda_stream"
PyObject *g_address_attr = nullptr;      // "_address"
PyTypeObject *g_desc_type = nullptr;     // binding.ConvDesc, from use_desc

struct Failed {};                        // a Python error is set

// One attribute of `o`, or of what it returns when called without arguments; a new reference.
PyObject *attribute(PyObject *o, const char *name, bool call)
{
    PyObject *v = call ? PyObject_CallMethod(o, name, nullptr) : PyObject_GetAttrString(o, name);
    if (!v) throw Failed();
    return v;
}

bool is_true(PyObject *o)
{
    const int v = PyObject_IsTrue(o);
    if (v < 0) throw Failed();
    return v != 0;
}

// The same for an object that is no torch.Tensor but answers as one (is_cuda, is_contiguous(), dtype, data_ptr()).
void *stand_in_ptr(PyObject *o, at::ScalarType type, const char *name)
{
    if (!PyObject_HasAttrString(o, "is_cuda")) {
        PyErr_Format(PyExc_TypeError, "%s must be a tensor", name);
        throw Failed();
    }
    const char *wrong = nullptr;
    PyObject *v = attribute(o, "is_cuda", false);
    if (!is_true(v)) wrong = "live in device memory";
    Py_DECREF(v);
    if (!wrong) {
        v = attribute(o, "is_contiguous", true);
        if (!is_true(v)) wrong = "be contiguous";
        Py_DECREF(v);
    }
    if (wrong) {
        PyErr_Format(PyExc_ValueError, "%s must %s", name, wrong);
        throw Failed();
    }
    v = attribute(o, "dtype", false);
    const int same = PyObject_RichCompareBool(v, (PyObject *)torch::getTHPDtype(type), Py_EQ);
    if (same == 0) PyErr_Format(PyExc_ValueError, "%s must have dtype %S, got %S", name, (PyObject *)torch::getTHPDtype(type), v);
    Py_DECREF(v);
    if (same != 1) throw Failed();
    v = attribute(o, "data_ptr", true);
    void *ptr = PyLong_AsVoidPtr(v);
    Py_DECREF(v);
    if (!ptr && PyErr_Occurred()) throw Failed();
    return ptr;
}

// The tensor's address; NULL for None.
void *device_ptr(PyObject *o, at::ScalarType type, const char *name)
{
    if (o == Py_None) return nullptr;
    if (!THPVariable_Check(o)) return stand_in_ptr(o, type, name);
    const at::Tensor &t = THPVariable_Unpack(o);
    const char *wrong = !t.is_cuda() ? "live in device memory" : (!t.is_contiguous() ? "be contiguous" : nullptr);
    if (wrong) {
        PyErr_Format(PyExc_ValueError, "%s must %s", name, wrong);
        throw Failed();
    }
    if (t.scalar_type() != type) {
        PyErr_Format(PyExc_ValueError, "%s must have dtype %S, got %S", name, (PyObject *)torch::getTHPDtype(type),
                     (PyObject *)torch::getTHPDtype(t.scalar_type()));
        throw Failed();
    }
    return t.data_ptr();
}

int64_t integer(PyObject *o)
{
    const int64_t v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw Failed();
    return v;
}

// Bytes of a buffer that device_ptr has checked.
size_t bytes_of(PyObject *o)
{
    if (o == Py_None) return 0;
    if (THPVariable_Check(o)) return (size_t)THPVariable_Unpack(o).numel();
    PyObject *v = attribute(o, "numel", true);
    const size_t n = PyLong_AsSize_t(v);
    Py_DECREF(v);
    if (n == (size_t)-1 && PyErr_Occurred()) throw Failed();
    return n;
}

double real(PyObject *o)
{
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) throw Failed();
    return v;
}

// hipStream_t of a torch stream; None: torch's current stream on the current device.
void *stream_of(PyObject *o)
{
    PyObject *value;
    if (o != Py_None) {
        value = PyObject_GetAttr(o, g_stream_attr);
    } else {
        PyObject *device = PyLong_FromLong(c10::impl::getDeviceGuardImpl(c10::DeviceType::CUDA)->getDevice().index());
        if (!device) throw Failed();
        value = PyObject_CallOneArg(g_raw_stream, device);
        Py_DECREF(device);
    }
    if (!value) throw Failed();
    void *s = PyLong_AsVoidPtr(value);
    Py_DECREF(value);
    if (!s && PyErr_Occurred()) throw Failed();
    return s;
}

// The convolution's geometry out of a binding.ConvDesc (a ctypes structure lends its memory as a buffer).
dg_conv_desc geometry(PyObject *o)
{
    if (!g_desc_type || !PyObject_TypeCheck(o, g_desc_type)) {
        PyErr_SetString(PyExc_TypeError, "desc must be a ConvDesc");
        throw Failed();
    }
    Py_buffer view;
    if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) throw Failed();
    dg_conv_desc d;
    const bool fits = view.len >= (Py_ssize_t)sizeof(d);
    if (fits) memcpy(&d, view.buf, sizeof(d));
    PyBuffer_Release(&view);
    if (!fits) {
        PyErr_SetString(PyExc_TypeError, "desc must be a ConvDesc");
        throw Failed();
    }
    return d;
}

// The table's address: a number, or a binding.Lut's, or the handle of another object that owns a table (a number or a ctypes
// pointer, whose value is None where it is NULL).
const dg_lut *table(PyObject *o)
{
    PyObject *address = nullptr;
    if (PyLong_Check(o)) {
        Py_INCREF(o);
        address = o;
    } else if (PyObject *own = PyObject_GetAttr(o, g_address_attr)) {
        address = own;
    } else {
        if (!PyErr_ExceptionMatches(PyExc_AttributeError)) throw Failed();
        PyErr_Clear();
        PyObject *handle = PyObject_GetAttrString(o, "handle");
        if (!handle) {
            PyErr_Format(PyExc_TypeError, "lut must be a table, got %.100s", Py_TYPE(o)->tp_name);
            throw Failed();
        }
        if (PyLong_Check(handle) || handle == Py_None) {
            address = handle;
        } else {
            address = PyObject_GetAttrString(handle, "value");
            Py_DECREF(handle);
            if (!address) throw Failed();
        }
    }
    const size_t value = address == Py_None ? 0 : PyLong_AsSize_t(address);
    Py_DECREF(address);
    if (value == (size_t)-1 && PyErr_Occurred()) throw Failed();
    return (const dg_lut *)value;
}

// Where the result goes: int32, or float32 with a scale or a binary32 table.
struct Output {
    int32_t *i = nullptr;
    float *f = nullptr;
    const float *scale = nullptr;
    Output(PyObject *out, PyObject *scale_o, PyObject *is_f32)
    {
        if (scale_o != Py_None || is_true(is_f32))
            f = (float *)device_ptr(out, at::kFloat, "out");
        else
            i = (int32_t *)device_ptr(out, at::kInt, "out");
        scale = (const float *)device_ptr(scale_o, at::kFloat, "scale");
    }
};

template <class Call>
PyObject *guarded(Py_ssize_t given, Py_ssize_t wanted, Call call)
{
    if (given != wanted) return PyErr_Format(PyExc_TypeError, "%zd arguments, %zd needed", given, wanted);
    try {
        return PyLong_FromLong((long)call());
    } catch (const Failed &) {
        return nullptr;
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

// The interpreter lock is away while one of these lives.
struct Unlocked {
    PyThreadState *const state = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(state); }
};

// EXPR: the library's call on values that are C's already, nothing of Python's.
#define RUN(EXPR)            \
    const Unlocked unlocked; \
    return EXPR

// (lut, is_f32, Wp, Xp, desc, out, scale, variant, stream)
PyObject *conv2d_lut(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 9, [&] {
        const dg_lut *lut = table(a[0]);
        const void *w = device_ptr(a[2], at::kByte, "Wp"), *x = device_ptr(a[3], at::kByte, "Xp");
        const dg_conv_desc d = geometry(a[4]);
        const Output o(a[5], a[6], a[1]);
        const dg_kernel variant = (dg_kernel)integer(a[7]);
        void *s = stream_of(a[8]);
        RUN(dg_conv2d_lut(lut, w, x, &d, o.i, o.scale, o.f, variant, s));
    });
}

// (lut, is_f32, Wp, Xc, desc, work, out, scale, variant, stream)
PyObject *conv2d_lut_codes(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 10, [&] {
        const dg_lut *lut = table(a[0]);
        const void *w = device_ptr(a[2], at::kByte, "Wp");
        const uint8_t *x = (const uint8_t *)device_ptr(a[3], at::kByte, "Xc");
        const dg_conv_desc d = geometry(a[4]);
        void *work = device_ptr(a[5], at::kByte, "work");
        const Output o(a[6], a[7], a[1]);
        const dg_kernel variant = (dg_kernel)integer(a[8]);
        void *s = stream_of(a[9]);
        const size_t bytes = bytes_of(a[5]);
        RUN(dg_conv2d_lut_codes(lut, w, x, &d, work, bytes, o.i, o.scale, o.f, variant, s));
    });
}

// (lut, is_f32, Wp, Xc, desc, out, scale, variant, stream)
PyObject *conv2d_lut_codes_static(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 9, [&] {
        const dg_lut *lut = table(a[0]);
        const void *w = device_ptr(a[2], at::kByte, "Wp");
        const uint8_t *x = (const uint8_t *)device_ptr(a[3], at::kByte, "Xc");
        const dg_conv_desc d = geometry(a[4]);
        const Output o(a[5], a[6], a[1]);
        const dg_kernel variant = (dg_kernel)integer(a[7]);
        void *s = stream_of(a[8]);
        RUN(dg_conv2d_lut_codes_static(lut, w, x, &d, o.i, o.scale, o.f, variant, s));
    });
}

// (lut, Wp, Xp, desc, scale, q_scale, q_zero, lo, out, variant, stream)
PyObject *conv2d_lut_requant(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 11, [&] {
        const dg_lut *lut = table(a[0]);
        const void *w = device_ptr(a[1], at::kByte, "Wp"), *x = device_ptr(a[2], at::kByte, "Xp");
        const dg_conv_desc d = geometry(a[3]);
        const float *scale = (const float *)device_ptr(a[4], at::kFloat, "scale");
        const float qs = (float)real(a[5]), qz = (float)real(a[6]);
        const int32_t lo = (int32_t)integer(a[7]);
        void *out = device_ptr(a[8], at::kByte, "packed");
        const dg_kernel variant = (dg_kernel)integer(a[9]);
        void *s = stream_of(a[10]);
        const size_t bytes = bytes_of(a[8]);
        RUN(dg_conv2d_lut_requant(lut, w, x, &d, scale, qs, qz, lo, out, bytes, variant, s));
    });
}

// (lut, is_f32, Wp, Ap, M, N, K, out, stride_m, stride_n, scale, variant, stream)
PyObject *gemm_lut(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 13, [&] {
        const dg_lut *lut = table(a[0]);
        const void *w = device_ptr(a[2], at::kByte, "Wp"), *x = device_ptr(a[3], at::kByte, "Ap");
        const int64_t M = integer(a[4]), N = integer(a[5]), K = integer(a[6]), sm = integer(a[8]), sn = integer(a[9]);
        const Output o(a[7], a[10], a[1]);
        const dg_kernel variant = (dg_kernel)integer(a[11]);
        void *s = stream_of(a[12]);
        RUN(dg_gemm_lut(lut, w, x, M, N, K, o.i, sm, sn, o.scale, o.f, variant, s));
    });
}

// (lut, is_f32, Wp, Ac, M, N, K, work, out, stride_m, stride_n, scale, variant, stream)
PyObject *gemm_lut_codes(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 14, [&] {
        const dg_lut *lut = table(a[0]);
        const void *w = device_ptr(a[2], at::kByte, "Wp");
        const uint8_t *x = (const uint8_t *)device_ptr(a[3], at::kByte, "Ac");
        const int64_t M = integer(a[4]), N = integer(a[5]), K = integer(a[6]), sm = integer(a[9]), sn = integer(a[10]);
        void *work = device_ptr(a[7], at::kByte, "work");
        const Output o(a[8], a[11], a[1]);
        const dg_kernel variant = (dg_kernel)integer(a[12]);
        void *s = stream_of(a[13]);
        const size_t bytes = bytes_of(a[7]);
        RUN(dg_gemm_lut_codes(lut, w, x, M, N, K, work, bytes, o.i, sm, sn, o.scale, o.f, variant, s));
    });
}

// (codes, rows, K, bits, out, stream)
PyObject *pack_codes_bits(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 6, [&] {
        const uint8_t *codes = (const uint8_t *)device_ptr(a[0], at::kByte, "codes");
        const int64_t rows = integer(a[1]), K = integer(a[2]);
        const int32_t bits = (int32_t)integer(a[3]);
        void *out = device_ptr(a[4], at::kByte, "packed");
        void *s = stream_of(a[5]);
        const size_t bytes = bytes_of(a[4]);
        RUN(dg_pack_codes_bits(codes, rows, K, bits, out, bytes, s));
    });
}

// (codes, rows, K, out, stream): weights, activations
template <dg_status (*FN)(const uint8_t *, int64_t, int64_t, void *, size_t, void *)>
PyObject *pack(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 5, [&] {
        const uint8_t *codes = (const uint8_t *)device_ptr(a[0], at::kByte, "codes");
        const int64_t rows = integer(a[1]), K = integer(a[2]);
        void *out = device_ptr(a[3], at::kByte, "packed");
        void *s = stream_of(a[4]);
        const size_t bytes = bytes_of(a[3]);
        RUN(FN(codes, rows, K, out, bytes, s));
    });
}

// (x, N, K, scale, zero_point, lo, out, stream)
PyObject *quantize_pack_activations(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 8, [&] {
        const float *x = (const float *)device_ptr(a[0], at::kFloat, "x");
        const int64_t N = integer(a[1]), K = integer(a[2]);
        const float scale = (float)real(a[3]), zero = (float)real(a[4]);
        const int32_t lo = (int32_t)integer(a[5]);
        void *out = device_ptr(a[6], at::kByte, "packed");
        void *s = stream_of(a[7]);
        const size_t bytes = bytes_of(a[6]);
        RUN(dg_quantize_pack_activations(x, N, K, scale, zero, lo, out, bytes, s));
    });
}

// (acc, rows, C, scale, out, stream)
PyObject *dequantize(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 6, [&] {
        const int32_t *acc = (const int32_t *)device_ptr(a[0], at::kInt, "acc");
        const int64_t rows = integer(a[1]), C = integer(a[2]);
        const float *scale = (const float *)device_ptr(a[3], at::kFloat, "scale");
        float *out = (float *)device_ptr(a[4], at::kFloat, "out");
        void *s = stream_of(a[5]);
        RUN(dg_dequantize(acc, rows, C, scale, out, s));
    });
}

// (type): binding.ConvDesc, whose instances alone are taken for a geometry
PyObject *use_desc(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 1, [&] {
        if (!PyType_Check(a[0])) {
            PyErr_SetString(PyExc_TypeError, "a type is needed");
            throw Failed();
        }
        Py_INCREF(a[0]);
        Py_XDECREF((PyObject *)g_desc_type);
        g_desc_type = (PyTypeObject *)a[0];
        return 0;
    });
}

#define METHOD(NAME, FN) {NAME, (PyCFunction)(void (*)(void))(FN), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    METHOD("conv2d_lut", conv2d_lut), METHOD("conv2d_lut_codes", conv2d_lut_codes),
    METHOD("conv2d_lut_codes_static", conv2d_lut_codes_static), METHOD("conv2d_lut_requant", conv2d_lut_requant),
    METHOD("gemm_lut", gemm_lut), METHOD("gemm_lut_codes", gemm_lut_codes), METHOD("pack_codes_bits", pack_codes_bits),
    METHOD("pack_weights", pack<dg_pack_weights>), METHOD("pack_activations", pack<dg_pack_activations>),
    METHOD("quantize_pack_activations", quantize_pack_activations), METHOD("dequantize", dequantize),
    METHOD("use_desc", use_desc),
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_native", "Tensors in, the C ABI's status out.", -1, methods,
                          nullptr, nullptr, nullptr, nullptr};

}   // namespace

PyMODINIT_FUNC PyInit__native()
{
    PyObject *torch_c = PyImport_ImportModule("torch._C");
    if (!torch_c) return nullptr;
    g_raw_stream = PyObject_GetAttrString(torch_c, "_cuda_getCurrentRawStream");
    Py_DECREF(torch_c);
    g_stream_attr = PyUnicode_InternFromString("cuda_stream");
    g_address_attr = PyUnicode_InternFromString("_address");
    if (!g_raw_stream || !g_stream_attr || !g_address_attr) return nullptr;
    return PyModule_Create(&module_def);
}
