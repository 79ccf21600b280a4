// The usual form of the short calls, checked and made without Python in between.
//
// A small layer is three calls of a few microseconds each on the GPU, and checking their tensors in Python and handing the
// arguments through ctypes took 2 to 2.6 us a call beside the 3.4 to 4.8 of the library's own entry (a launch is 2.4).  Each
// function here takes the tensors of one public call, all of its outputs among them, asks what binding.py asks of them, and
// calls the C entry: 64 x 256 x 256 as three calls 20.3 -> 11.1 us, which is what their kernels take.  Whatever is not the
// plain case (a subclass, a wrong type or shape, another device, an output that has to be allocated) is not decided here:
// kNotPlain, after 0.1 us, sends the caller through the checks in binding.py, which say what is wrong or make the call.
// Nothing is kept from one call for the next.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/crossquant.h"

namespace {

constexpr int kNotPlain = 1;             // no status of the library is positive

// The C entries, by the addresses that binding.py hands over: the library that it has loaded is the one that is called.
decltype(&crossquant_absmax) p_absmax;
decltype(&crossquant_quantize) p_quantize;
decltype(&crossquant_absmax_quantize) p_absmax_quantize;
decltype(&crossquant_quantize_fp6) p_quantize_fp6;
decltype(&crossquant_absmax_batched) p_absmax_batched;
decltype(&crossquant_quantize_batched) p_quantize_batched;
decltype(&crossquant_kernel_count) p_kernel_count;
decltype(&crossquant_kernel_analysis) p_kernel_analysis;
decltype(&crossquant_w8a8_linear) p_w8a8_linear;
decltype(&crossquant_w4a4_linear) p_w4a4_linear;
decltype(&crossquant_fp6_packed_bytes) p_fp6_packed_bytes;
decltype(&crossquant_fp6_packed_weight_bytes) p_fp6_packed_weight_bytes;

// The questions below answer false for what is not plain and leave their results unset.  (No exceptions: one costs as much as the
// whole Python check, 4.6 us against 0.1 for a refused w8a8_linear.)

// a tensor or a parameter; other subclasses have their own ideas
bool tensor(PyObject* o, const at::Tensor*& t) {
    if (!THPVariable_CheckExact(o)) return false;
    t = &THPVariable_Unpack(o);
    return true;
}

bool is(const at::Tensor& t, at::ScalarType type, c10::DeviceIndex device) {
    return t.scalar_type() == type && t.is_cuda() && t.get_device() == device;
}

// the leading operand: a 2-D GPU tensor with unit stride along rows that do not overlap
struct Matrix {
    const at::Tensor* t;
    int64_t rows, cols, ld;
    c10::DeviceIndex device;
    void* data;
    void* stream() const { return c10::hip::getCurrentHIPStream(device).stream(); }
};
bool matrix(PyObject* o, at::ScalarType type, Matrix& X) {
    if (!tensor(o, X.t) || X.t->scalar_type() != type || X.t->dim() != 2 || !X.t->is_cuda()) return false;
    X.rows = X.t->size(0);
    X.cols = X.t->size(1);
    X.ld = X.t->stride(0);
    if (X.t->stride(1) != 1 || X.ld < X.cols) return false;
    X.device = X.t->get_device();
    X.data = X.t->data_ptr();
    return true;
}

template <typename P>
bool buffer(PyObject* o, P*& p, at::ScalarType type, c10::DeviceIndex device, int64_t n0, int64_t n1 = -1) {
    const at::Tensor* t;
    if (!tensor(o, t) || !is(*t, type, device) || !t->is_contiguous()) return false;
    if (n1 < 0 ? (t->dim() != 1 || t->size(0) != n0) : (t->dim() != 2 || t->size(0) != n0 || t->size(1) != n1)) return false;
    p = static_cast<P*>(t->data_ptr());
    return true;
}
template <typename P>
bool optional_buffer(PyObject* o, P*& p, at::ScalarType type, c10::DeviceIndex device, int64_t n0, int64_t n1 = -1) {
    p = nullptr;
    return o == Py_None || buffer(o, p, type, device, n0, n1);
}
template <typename P>                    // (float or const float)
bool floats(PyObject* o, P*& p, c10::DeviceIndex device, int64_t n) { return buffer(o, p, at::kFloat, device, n); }

bool integer(PyObject* o, int64_t& v) {
    if (!PyLong_CheckExact(o)) return false;
    int overflow;
    v = PyLong_AsLongLongAndOverflow(o, &overflow);
    return !overflow;
}
// alpha, also as an integer
bool real(PyObject* o, float& v) {
    int64_t whole;
    if (PyFloat_CheckExact(o)) v = (float)PyFloat_AS_DOUBLE(o);
    else if (integer(o, whole)) v = (float)(double)whole;
    else return false;
    return true;
}
bool bits_of(PyObject* o, int64_t cols, int& bits) {
    int64_t v;
    if (!integer(o, v) || (v != 8 && (v != 4 || cols % 2))) return false;
    bits = (int)v;
    return true;
}
bool codes_of(PyObject* o, const Matrix& X, int bits, void*& p) {
    return bits == 8 ? buffer(o, p, at::kChar, X.device, X.rows, X.cols) : buffer(o, p, at::kByte, X.device, X.rows, X.cols / 2);
}
// an output of T rows of O values that may be padded
bool output(PyObject* o, c10::DeviceIndex device, int64_t T, int64_t O, void*& p, int64_t& ldy) {
    const at::Tensor* t;
    if (!tensor(o, t) || !is(*t, at::kHalf, device) || t->dim() != 2 || t->size(0) != T || t->size(1) != O) return false;
    ldy = t->stride(0);
    if (t->stride(1) != 1 || ldy < O) return false;
    p = t->data_ptr();
    return true;
}

// the C entry without the interpreter's lock, as ctypes calls it
template <typename F>
int unlocked(F&& f) {
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = f();
    Py_END_ALLOW_THREADS
    return status;
}

// N arguments, a status back; what torch throws on the way, for instance for a tensor without storage, is for the Python checks
// to say
template <int N, typename F>
PyObject* call(Py_ssize_t n, F&& f) {
    if (n != N) {
        PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
        return nullptr;
    }
    int status = kNotPlain;
    try {
        status = f();
    } catch (...) {
        PyErr_Clear();
    }
    return PyLong_FromLong(status);
}

PyObject* absmax(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return call<3>(n, [&] {
        Matrix X;
        float *t, *c;
        if (!matrix(a[0], at::kHalf, X) || !floats(a[1], t, X.device, X.rows) || !floats(a[2], c, X.device, X.cols)) return kNotPlain;
        void* s = X.stream();
        return unlocked([&] { return p_absmax(X.data, X.rows, X.cols, X.ld, t, c, s); });
    });
}

// X, t, c, alpha, bits, codes, xhat or None, row_scale, col_scale, zero_count or None
PyObject* quantize(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return call<10>(n, [&] {
        Matrix X;
        const float *t, *c;
        float alpha, *rs, *cs;
        int bits;
        void *codes, *xhat;
        unsigned long long* z;
        if (!matrix(a[0], at::kHalf, X) || !floats(a[1], t, X.device, X.rows) || !floats(a[2], c, X.device, X.cols) || !real(a[3], alpha) ||
            !bits_of(a[4], X.cols, bits) || !codes_of(a[5], X, bits, codes) || !optional_buffer(a[6], xhat, at::kHalf, X.device, X.rows, X.cols) ||
            !floats(a[7], rs, X.device, X.rows) || !floats(a[8], cs, X.device, X.cols) || !optional_buffer(a[9], z, at::kLong, X.device, 1))
            return kNotPlain;
        void* s = X.stream();
        return unlocked([&] { return p_quantize(X.data, X.rows, X.cols, X.ld, t, c, alpha, bits, codes, xhat, rs, cs, z, s); });
    });
}

// X, alpha, bits, t, c, codes, xhat or None, row_scale, col_scale, zero_count or None
PyObject* absmax_quantize(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return call<10>(n, [&] {
        Matrix X;
        float alpha, *t, *c, *rs, *cs;
        int bits;
        void *codes, *xhat;
        unsigned long long* z;
        if (!matrix(a[0], at::kHalf, X) || !real(a[1], alpha) || !bits_of(a[2], X.cols, bits) || !floats(a[3], t, X.device, X.rows) ||
            !floats(a[4], c, X.device, X.cols) || !codes_of(a[5], X, bits, codes) || !optional_buffer(a[6], xhat, at::kHalf, X.device, X.rows, X.cols) ||
            !floats(a[7], rs, X.device, X.rows) || !floats(a[8], cs, X.device, X.cols) || !optional_buffer(a[9], z, at::kLong, X.device, 1))
            return kNotPlain;
        void* s = X.stream();
        return unlocked([&] { return p_absmax_quantize(X.data, X.rows, X.cols, X.ld, alpha, bits, t, c, codes, xhat, rs, cs, z, s); });
    });
}

// X, t, c, alpha, packed, xhat or None, row_scale, col_scale, zero_count or None
PyObject* quantize_fp6(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return call<9>(n, [&] {
        Matrix X;
        const float *t, *c;
        float alpha, *rs, *cs;
        void *packed, *xhat;
        unsigned long long* z;
        if (!matrix(a[0], at::kHalf, X)) return kNotPlain;
        const int64_t bytes = p_fp6_packed_bytes(X.rows, X.cols);
        if (bytes < 0 || !floats(a[1], t, X.device, X.rows) || !floats(a[2], c, X.device, X.cols) || !real(a[3], alpha) ||
            !buffer(a[4], packed, at::kByte, X.device, bytes) || !optional_buffer(a[5], xhat, at::kHalf, X.device, X.rows, X.cols) ||
            !floats(a[6], rs, X.device, X.rows) || !floats(a[7], cs, X.device, X.cols) || !optional_buffer(a[8], z, at::kLong, X.device, 1))
            return kNotPlain;
        void* s = X.stream();
        return unlocked([&] { return p_quantize_fp6(X.data, X.rows, X.cols, X.ld, t, c, alpha, packed, xhat, rs, cs, z, s); });
    });
}

// a [B][S][I] GPU tensor with contiguous rows
struct Batch {
    const at::Tensor* t;
    int64_t B, S, I, ld, step;
    c10::DeviceIndex device;
    void* data;
    void* stream() const { return c10::hip::getCurrentHIPStream(device).stream(); }
};
bool batch(PyObject* o, Batch& X) {
    if (!tensor(o, X.t) || X.t->scalar_type() != at::kHalf || X.t->dim() != 3 || !X.t->is_cuda()) return false;
    X.B = X.t->size(0);
    X.S = X.t->size(1);
    X.I = X.t->size(2);
    if (X.t->stride(2) != 1 && X.I != 1) return false;
    X.ld = X.t->stride(1);
    X.step = X.t->stride(0);
    X.device = X.t->get_device();
    X.data = X.t->data_ptr();
    return true;
}

PyObject* absmax_batched(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return call<3>(n, [&] {
        Batch X;
        float *t, *c;
        if (!batch(a[0], X) || !buffer(a[1], t, at::kFloat, X.device, X.B, X.S) || !buffer(a[2], c, at::kFloat, X.device, X.B, X.I)) return kNotPlain;
        void* s = X.stream();
        return unlocked([&] { return p_absmax_batched(X.data, X.B, X.S, X.I, X.ld, X.step, t, c, s); });
    });
}

// X, t, c, alpha, bits, codes?, xhat?, count? -> the five outputs, allocated here (codes, xhat and count or None), or a status
PyObject* quantize_batched(PyObject*, PyObject* const* a, Py_ssize_t n) {
    at::Tensor codes, xhat, rs, cs, z;
    PyObject* status = call<8>(n, [&] {
        Batch X;
        float alpha;
        int bits;
        if (!batch(a[0], X) || !real(a[3], alpha) || !bits_of(a[4], X.I, bits)) return kNotPlain;
        for (int i = 5; i < 8; ++i)
            if (a[i] != Py_True && a[i] != Py_False) return kNotPlain;
        const bool want_codes = a[5] == Py_True, want_xhat = a[6] == Py_True && want_codes, want_count = a[7] == Py_True || !want_codes;
        const float* in[2];                                  // any shape that holds as many values
        for (int i = 0; i < 2; ++i) {
            const at::Tensor* v;
            if (!tensor(a[1 + i], v) || !is(*v, at::kFloat, X.device) || !v->is_contiguous() || v->numel() != X.B * (i ? X.I : X.S)) return kNotPlain;
            in[i] = static_cast<const float*>(v->data_ptr());
        }
        auto empty = [&](at::IntArrayRef shape, at::ScalarType type) { return at::empty(shape, at::TensorOptions().dtype(type).device(X.t->device())); };
        if (want_codes) codes = bits == 8 ? empty({X.B, X.S, X.I}, at::kChar) : empty({X.B, X.S, X.I / 2}, at::kByte);
        if (want_xhat) xhat = empty({X.B, X.S, X.I}, at::kHalf);
        rs = empty({X.B, X.S}, at::kFloat);
        cs = empty({X.B, X.I}, at::kFloat);
        if (want_count) z = empty({1}, at::kLong);
        void *codes_p = want_codes ? codes.data_ptr() : nullptr, *xhat_p = want_xhat ? xhat.data_ptr() : nullptr;
        auto *rs_p = static_cast<float*>(rs.data_ptr()), *cs_p = static_cast<float*>(cs.data_ptr());
        auto* z_p = want_count ? static_cast<unsigned long long*>(z.data_ptr()) : nullptr;
        void* s = X.stream();
        return unlocked([&] { return p_quantize_batched(X.data, X.B, X.S, X.I, X.ld, X.step, in[0], in[1], alpha, bits, codes_p, xhat_p, rs_p, cs_p, z_p, s); });
    });
    if (!status || PyLong_AsLong(status) != 0) return status;
    Py_DECREF(status);
    PyObject* out = PyTuple_New(5);
    if (!out) return nullptr;
    const at::Tensor* const tensors[] = {&codes, &xhat, &rs, &cs, &z};
    for (int i = 0; i < 5; ++i) {
        PyObject* o = tensors[i]->defined() ? THPVariable_Wrap(*tensors[i]) : (Py_INCREF(Py_None), Py_None);
        if (!o) {
            Py_DECREF(out);
            return nullptr;
        }
        PyTuple_SET_ITEM(out, i, o);
    }
    return out;
}

// 4 or 8 for the calls that write no codes, whatever the number of channels
bool count_bits(PyObject* o, int& bits) { return bits_of(o, 0, bits); }

// X, t, c, alpha, bits, row_scale and col_scale or None, zero_count
PyObject* kernel_count(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return call<8>(n, [&] {
        Matrix X;
        const float *t, *c;
        float alpha, *rs, *cs;
        int bits;
        unsigned long long* z;
        if (!matrix(a[0], at::kHalf, X) || !floats(a[1], t, X.device, X.rows) || !floats(a[2], c, X.device, X.cols) || !real(a[3], alpha) ||
            !count_bits(a[4], bits) || (a[5] == Py_None) != (a[6] == Py_None) || !optional_buffer(a[5], rs, at::kFloat, X.device, X.rows) ||
            !optional_buffer(a[6], cs, at::kFloat, X.device, X.cols) || !buffer(a[7], z, at::kLong, X.device, 1))
            return kNotPlain;
        void* s = X.stream();
        return unlocked([&] { return p_kernel_count(X.data, X.rows, X.cols, X.ld, t, c, alpha, bits, rs, cs, z, s); });
    });
}

// X, t, c, alpha, bits, xrk or None, row_scale and col_scale or None, counters
PyObject* kernel_analysis(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return call<9>(n, [&] {
        Matrix X;
        const float *t, *c;
        float alpha, *rs, *cs;
        int bits;
        void* xrk;
        unsigned long long* counters;
        if (!matrix(a[0], at::kHalf, X) || !floats(a[1], t, X.device, X.rows) || !floats(a[2], c, X.device, X.cols) || !real(a[3], alpha) ||
            !count_bits(a[4], bits) || !optional_buffer(a[5], xrk, at::kHalf, X.device, X.rows, X.cols) || (a[6] == Py_None) != (a[7] == Py_None) ||
            !optional_buffer(a[6], rs, at::kFloat, X.device, X.rows) || !optional_buffer(a[7], cs, at::kFloat, X.device, X.cols) ||
            !buffer(a[8], counters, at::kLong, X.device, 3))
            return kNotPlain;
        void* s = X.stream();
        return unlocked([&] { return p_kernel_analysis(X.data, X.rows, X.cols, X.ld, t, c, alpha, bits, xrk, rs, cs, counters, s); });
    });
}

// qx, row_scale, qw, w_scale, Y
PyObject* w8a8_linear(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return call<5>(n, [&] {
        Matrix qx, qw;
        const float *rs, *ws;
        void* Y;
        int64_t ldy;
        if (!matrix(a[0], at::kChar, qx) || !matrix(a[2], at::kChar, qw) || !qx.t->is_contiguous() || !qw.t->is_contiguous() ||
            qx.cols != qw.cols || qw.device != qx.device || !floats(a[1], rs, qx.device, qx.rows) || !floats(a[3], ws, qx.device, qw.rows) ||
            !output(a[4], qx.device, qx.rows, qw.rows, Y, ldy))
            return kNotPlain;
        void* s = qx.stream();
        return unlocked([&] {
            return p_w8a8_linear(static_cast<const int8_t*>(qx.data), rs, static_cast<const int8_t*>(qw.data), ws, qx.rows, qx.cols, qw.rows, Y, ldy, nullptr, s);
        });
    });
}

// qx_fp6, row_scale, qw_fp6, w_scale, T, I, O, Y
PyObject* w4a4_linear(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return call<8>(n, [&] {
        const at::Tensor* q[2];
        int64_t T, I, O, ldy;
        const float *rs, *ws;
        void* Y;
        if (!tensor(a[0], q[0]) || !tensor(a[2], q[1]) || !q[0]->is_cuda() || !integer(a[4], T) || !integer(a[5], I) || !integer(a[6], O))
            return kNotPlain;
        const c10::DeviceIndex device = q[0]->get_device();
        for (int i = 0; i < 2; ++i)
            if (!is(*q[i], at::kByte, device) || !q[i]->is_contiguous() ||
                q[i]->numel() != (i ? p_fp6_packed_weight_bytes(O, I) : p_fp6_packed_bytes(T, I))) return kNotPlain;
        if (!floats(a[1], rs, device, T) || !floats(a[3], ws, device, O) || !output(a[7], device, T, O, Y, ldy)) return kNotPlain;
        const void *x = q[0]->data_ptr(), *w = q[1]->data_ptr();
        void* s = c10::hip::getCurrentHIPStream(device).stream();
        return unlocked([&] { return p_w4a4_linear(x, rs, w, ws, T, I, O, Y, ldy, nullptr, s); });
    });
}

// the addresses of the C entries, in the order of the pointers above
PyObject* set_entries(PyObject*, PyObject* const* a, Py_ssize_t n) {
    void** const entries[] = {reinterpret_cast<void**>(&p_absmax), reinterpret_cast<void**>(&p_quantize),
                              reinterpret_cast<void**>(&p_absmax_quantize), reinterpret_cast<void**>(&p_quantize_fp6),
                              reinterpret_cast<void**>(&p_absmax_batched), reinterpret_cast<void**>(&p_quantize_batched),
                              reinterpret_cast<void**>(&p_kernel_count), reinterpret_cast<void**>(&p_kernel_analysis),
                              reinterpret_cast<void**>(&p_w8a8_linear), reinterpret_cast<void**>(&p_w4a4_linear),
                              reinterpret_cast<void**>(&p_fp6_packed_bytes), reinterpret_cast<void**>(&p_fp6_packed_weight_bytes)};
    constexpr Py_ssize_t kEntries = sizeof(entries) / sizeof(entries[0]);
    if (n != kEntries) {
        PyErr_SetString(PyExc_TypeError, "wrong number of entries");
        return nullptr;
    }
    for (Py_ssize_t i = 0; i < n; ++i) {
        void* p = PyLong_AsVoidPtr(a[i]);
        if (!p) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "a null entry");
            return nullptr;
        }
        *entries[i] = p;
    }
    Py_RETURN_NONE;
}

#define CQ_METHOD(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&f)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {CQ_METHOD(absmax_batched),  CQ_METHOD(quantize_batched),
                         CQ_METHOD(absmax),          CQ_METHOD(quantize),    CQ_METHOD(absmax_quantize), CQ_METHOD(quantize_fp6), CQ_METHOD(kernel_count),
                         CQ_METHOD(kernel_analysis), CQ_METHOD(w8a8_linear), CQ_METHOD(w4a4_linear),     CQ_METHOD(set_entries),  {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall() {
    PyObject* m = PyModule_Create(&module);
    if (m && (PyModule_AddIntConstant(m, "NOT_PLAIN", kNotPlain) < 0 || PyModule_AddStringConstant(m, "TORCH_VERSION", CQ_TORCH_VERSION) < 0)) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
