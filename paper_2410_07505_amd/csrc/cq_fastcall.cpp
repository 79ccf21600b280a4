// The usual form of the short calls, checked and made without Python in between.
//
// A small layer is three calls of a few microseconds each on the GPU, and checking their tensors in Python and handing the
// arguments through ctypes took 2 to 2.6 us a call beside the 3.4 to 4.8 of the library's own entry (a launch is 2.4).  Each
// function here takes the tensors of one public call, all of its outputs among them, asks what binding.py asks of them, and
// calls the C entry: 64 x 256 x 256 as
// three calls 20.3 -> 11.1 us, which is what their kernels take.  Whatever is not the plain case (a subclass, a wrong type or
// shape, another device, an output that has to be allocated) is not decided here: kNotPlain sends the caller through the checks
// in binding.py, which say what is wrong or make the call.  Nothing is kept from one call for the next.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/crossquant.h"

namespace {

constexpr int kNotPlain = 1;             // no status of the library is positive

struct NotPlain {};

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

const at::Tensor& tensor(PyObject* o) {
    if (Py_TYPE(o) != reinterpret_cast<PyTypeObject*>(THPVariableClass)) throw NotPlain{};      // subclasses have their own ideas
    return THPVariable_Unpack(o);
}

// the leading operand: a 2-D GPU tensor with unit stride along rows that do not overlap
struct Matrix {
    const at::Tensor& t;
    int64_t rows, cols, ld;
    c10::DeviceIndex device;
    void* data;
    Matrix(PyObject* o, at::ScalarType type) : t(tensor(o)) {
        if (t.scalar_type() != type || t.dim() != 2 || !t.is_cuda()) throw NotPlain{};
        rows = t.size(0);
        cols = t.size(1);
        ld = t.stride(0);
        if (t.stride(1) != 1 || ld < cols) throw NotPlain{};
        device = t.get_device();
        data = t.data_ptr();
    }
    void* stream() const { return c10::hip::getCurrentHIPStream(device).stream(); }
};

void* buffer(PyObject* o, at::ScalarType type, c10::DeviceIndex device, int64_t n0, int64_t n1 = -1) {
    const at::Tensor& t = tensor(o);
    if (t.scalar_type() != type || !t.is_cuda() || t.get_device() != device || !t.is_contiguous()) throw NotPlain{};
    if (n1 < 0 ? (t.dim() != 1 || t.size(0) != n0) : (t.dim() != 2 || t.size(0) != n0 || t.size(1) != n1)) throw NotPlain{};
    return t.data_ptr();
}
void* optional_buffer(PyObject* o, at::ScalarType type, c10::DeviceIndex device, int64_t n0, int64_t n1 = -1) {
    return o == Py_None ? nullptr : buffer(o, type, device, n0, n1);
}
float* floats(PyObject* o, c10::DeviceIndex device, int64_t n) { return static_cast<float*>(buffer(o, at::kFloat, device, n)); }

int64_t integer(PyObject* o) {
    if (!PyLong_CheckExact(o)) throw NotPlain{};
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw NotPlain{};
    return v;
}
float real(PyObject* o) {
    if (!PyFloat_CheckExact(o)) throw NotPlain{};
    return (float)PyFloat_AS_DOUBLE(o);
}
int bits_of(PyObject* o, int64_t cols) {
    const int64_t bits = integer(o);
    if (bits != 8 && (bits != 4 || cols % 2)) throw NotPlain{};
    return (int)bits;
}
void* codes_of(PyObject* o, const Matrix& X, int bits) {
    return bits == 8 ? buffer(o, at::kChar, X.device, X.rows, X.cols) : buffer(o, at::kByte, X.device, X.rows, X.cols / 2);
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

// N arguments, a status back; whatever is thrown on the way -- NotPlain, or torch's own errors, for instance for a tensor without
// storage -- is for the Python checks to say
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
        const Matrix X(a[0], at::kHalf);
        float *t = floats(a[1], X.device, X.rows), *c = floats(a[2], X.device, X.cols);
        void* s = X.stream();
        return unlocked([&] { return p_absmax(X.data, X.rows, X.cols, X.ld, t, c, s); });
    });
}

// X, t, c, alpha, bits, codes, xhat or None, row_scale, col_scale, zero_count or None
PyObject* quantize(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return call<10>(n, [&] {
        const Matrix X(a[0], at::kHalf);
        const float *t = floats(a[1], X.device, X.rows), *c = floats(a[2], X.device, X.cols), alpha = real(a[3]);
        const int bits = bits_of(a[4], X.cols);
        void *codes = codes_of(a[5], X, bits), *xhat = optional_buffer(a[6], at::kHalf, X.device, X.rows, X.cols);
        float *rs = floats(a[7], X.device, X.rows), *cs = floats(a[8], X.device, X.cols);
        auto* z = static_cast<unsigned long long*>(optional_buffer(a[9], at::kLong, X.device, 1));
        void* s = X.stream();
        return unlocked([&] { return p_quantize(X.data, X.rows, X.cols, X.ld, t, c, alpha, bits, codes, xhat, rs, cs, z, s); });
    });
}

// X, alpha, bits, t, c, codes, xhat or None, row_scale, col_scale, zero_count or None
PyObject* absmax_quantize(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return call<10>(n, [&] {
        const Matrix X(a[0], at::kHalf);
        const float alpha = real(a[1]);
        const int bits = bits_of(a[2], X.cols);
        float *t = floats(a[3], X.device, X.rows), *c = floats(a[4], X.device, X.cols);
        void *codes = codes_of(a[5], X, bits), *xhat = optional_buffer(a[6], at::kHalf, X.device, X.rows, X.cols);
        float *rs = floats(a[7], X.device, X.rows), *cs = floats(a[8], X.device, X.cols);
        auto* z = static_cast<unsigned long long*>(optional_buffer(a[9], at::kLong, X.device, 1));
        void* s = X.stream();
        return unlocked([&] { return p_absmax_quantize(X.data, X.rows, X.cols, X.ld, alpha, bits, t, c, codes, xhat, rs, cs, z, s); });
    });
}

// X, t, c, alpha, packed, xhat or None, row_scale, col_scale, zero_count or None
PyObject* quantize_fp6(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return call<9>(n, [&] {
        const Matrix X(a[0], at::kHalf);
        const int64_t bytes = p_fp6_packed_bytes(X.rows, X.cols);
        if (bytes < 0) throw NotPlain{};
        const float *t = floats(a[1], X.device, X.rows), *c = floats(a[2], X.device, X.cols), alpha = real(a[3]);
        void *packed = buffer(a[4], at::kByte, X.device, bytes), *xhat = optional_buffer(a[5], at::kHalf, X.device, X.rows, X.cols);
        float *rs = floats(a[6], X.device, X.rows), *cs = floats(a[7], X.device, X.cols);
        auto* z = static_cast<unsigned long long*>(optional_buffer(a[8], at::kLong, X.device, 1));
        void* s = X.stream();
        return unlocked([&] { return p_quantize_fp6(X.data, X.rows, X.cols, X.ld, t, c, alpha, packed, xhat, rs, cs, z, s); });
    });
}

// a [B][S][I] GPU tensor with contiguous rows
struct Batch {
    const at::Tensor& t;
    int64_t B, S, I;
    c10::DeviceIndex device;
    explicit Batch(PyObject* o) : t(tensor(o)) {
        if (t.scalar_type() != at::kHalf || t.dim() != 3 || !t.is_cuda()) throw NotPlain{};
        B = t.size(0);
        S = t.size(1);
        I = t.size(2);
        if (t.stride(2) != 1 && I != 1) throw NotPlain{};
        device = t.get_device();
    }
};

PyObject* absmax_batched(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return call<3>(n, [&] {
        const Batch X(a[0]);
        auto *t = static_cast<float*>(buffer(a[1], at::kFloat, X.device, X.B, X.S)), *c = static_cast<float*>(buffer(a[2], at::kFloat, X.device, X.B, X.I));
        const void* x = X.t.data_ptr();
        const int64_t ld = X.t.stride(1), step = X.t.stride(0);
        void* s = c10::hip::getCurrentHIPStream(X.device).stream();
        return unlocked([&] { return p_absmax_batched(x, X.B, X.S, X.I, ld, step, t, c, s); });
    });
}

// X, t, c, alpha, bits, codes?, xhat?, count? -> the five outputs, allocated here (codes, xhat and count or None), or a status
PyObject* quantize_batched(PyObject*, PyObject* const* a, Py_ssize_t n) {
    at::Tensor codes, xhat, rs, cs, z;
    PyObject* status = call<8>(n, [&] {
        const Batch X(a[0]);
        const at::Tensor &t = tensor(a[1]), &c = tensor(a[2]);
        const float alpha = real(a[3]);
        const int64_t bits = integer(a[4]);
        const bool want_codes = a[5] == Py_True, want_xhat = a[6] == Py_True && want_codes, want_count = a[7] == Py_True || !want_codes;
        for (int i = 5; i < 8; ++i)
            if (a[i] != Py_True && a[i] != Py_False) throw NotPlain{};
        if (bits != 8 && (bits != 4 || X.I % 2)) throw NotPlain{};
        for (const at::Tensor* v : {&t, &c})
            if (v->scalar_type() != at::kFloat || !v->is_cuda() || v->get_device() != X.device || !v->is_contiguous() ||
                v->numel() != X.B * (v == &t ? X.S : X.I)) throw NotPlain{};
        auto empty = [&](at::IntArrayRef shape, at::ScalarType type) { return at::empty(shape, at::TensorOptions().dtype(type).device(X.t.device())); };
        if (want_codes) codes = bits == 8 ? empty({X.B, X.S, X.I}, at::kChar) : empty({X.B, X.S, X.I / 2}, at::kByte);
        if (want_xhat) xhat = empty({X.B, X.S, X.I}, at::kHalf);
        rs = empty({X.B, X.S}, at::kFloat);
        cs = empty({X.B, X.I}, at::kFloat);
        if (want_count) z = empty({1}, at::kLong);
        const void* x = X.t.data_ptr();
        const int64_t ld = X.t.stride(1), step = X.t.stride(0);
        const auto *tp = static_cast<const float*>(t.data_ptr()), *cp = static_cast<const float*>(c.data_ptr());
        void *codes_p = want_codes ? codes.data_ptr() : nullptr, *xhat_p = want_xhat ? xhat.data_ptr() : nullptr;
        auto *rs_p = static_cast<float*>(rs.data_ptr()), *cs_p = static_cast<float*>(cs.data_ptr());
        auto* z_p = want_count ? static_cast<unsigned long long*>(z.data_ptr()) : nullptr;
        void* s = c10::hip::getCurrentHIPStream(X.device).stream();
        return unlocked([&] { return p_quantize_batched(x, X.B, X.S, X.I, ld, step, tp, cp, alpha, (int)bits, codes_p, xhat_p, rs_p, cs_p, z_p, s); });
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

// X, t, c, alpha, bits, row_scale and col_scale or None, zero_count
PyObject* kernel_count(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return call<8>(n, [&] {
        const Matrix X(a[0], at::kHalf);
        const float *t = floats(a[1], X.device, X.rows), *c = floats(a[2], X.device, X.cols), alpha = real(a[3]);
        const int64_t bits = integer(a[4]);
        if (bits != 4 && bits != 8) throw NotPlain{};
        if ((a[5] == Py_None) != (a[6] == Py_None)) throw NotPlain{};
        auto* rs = static_cast<float*>(optional_buffer(a[5], at::kFloat, X.device, X.rows));
        auto* cs = static_cast<float*>(optional_buffer(a[6], at::kFloat, X.device, X.cols));
        auto* z = static_cast<unsigned long long*>(buffer(a[7], at::kLong, X.device, 1));
        void* s = X.stream();
        return unlocked([&] { return p_kernel_count(X.data, X.rows, X.cols, X.ld, t, c, alpha, (int)bits, rs, cs, z, s); });
    });
}

// X, t, c, alpha, bits, xrk or None, row_scale and col_scale or None, counters
PyObject* kernel_analysis(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return call<9>(n, [&] {
        const Matrix X(a[0], at::kHalf);
        const float *t = floats(a[1], X.device, X.rows), *c = floats(a[2], X.device, X.cols), alpha = real(a[3]);
        const int64_t bits = integer(a[4]);
        if (bits != 4 && bits != 8) throw NotPlain{};
        void* xrk = optional_buffer(a[5], at::kHalf, X.device, X.rows, X.cols);
        if ((a[6] == Py_None) != (a[7] == Py_None)) throw NotPlain{};
        auto* rs = static_cast<float*>(optional_buffer(a[6], at::kFloat, X.device, X.rows));
        auto* cs = static_cast<float*>(optional_buffer(a[7], at::kFloat, X.device, X.cols));
        auto* counters = static_cast<unsigned long long*>(buffer(a[8], at::kLong, X.device, 3));
        void* s = X.stream();
        return unlocked([&] { return p_kernel_analysis(X.data, X.rows, X.cols, X.ld, t, c, alpha, (int)bits, xrk, rs, cs, counters, s); });
    });
}

// qx, row_scale, qw, w_scale, Y (contiguous)
PyObject* w8a8_linear(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return call<5>(n, [&] {
        const Matrix qx(a[0], at::kChar), qw(a[2], at::kChar);
        if (!qx.t.is_contiguous() || !qw.t.is_contiguous() || qx.cols != qw.cols || qw.device != qx.device) throw NotPlain{};
        const float *rs = floats(a[1], qx.device, qx.rows), *ws = floats(a[3], qx.device, qw.rows);
        void* Y = buffer(a[4], at::kHalf, qx.device, qx.rows, qw.rows);
        const int64_t ldy = THPVariable_Unpack(a[4]).stride(0);
        void* s = qx.stream();
        return unlocked([&] {
            return p_w8a8_linear(static_cast<const int8_t*>(qx.data), rs, static_cast<const int8_t*>(qw.data), ws, qx.rows, qx.cols, qw.rows, Y, ldy, nullptr, s);
        });
    });
}

// qx_fp6, row_scale, qw_fp6, w_scale, T, I, O, Y (contiguous)
PyObject* w4a4_linear(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return call<8>(n, [&] {
        const int64_t T = integer(a[4]), I = integer(a[5]), O = integer(a[6]);
        const at::Tensor &qx = tensor(a[0]), &qw = tensor(a[2]);
        if (!qx.is_cuda()) throw NotPlain{};
        const c10::DeviceIndex device = qx.get_device();
        for (const at::Tensor* q : {&qx, &qw})
            if (q->scalar_type() != at::kByte || !q->is_cuda() || q->get_device() != device || !q->is_contiguous()) throw NotPlain{};
        if (qx.numel() != p_fp6_packed_bytes(T, I) || qw.numel() != p_fp6_packed_weight_bytes(O, I)) throw NotPlain{};
        const float *rs = floats(a[1], device, T), *ws = floats(a[3], device, O);
        void* Y = buffer(a[7], at::kHalf, device, T, O);
        const int64_t ldy = THPVariable_Unpack(a[7]).stride(0);
        const void *x = qx.data_ptr(), *w = qw.data_ptr();
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
    if (m && PyModule_AddIntConstant(m, "NOT_PLAIN", kNotPlain) < 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
