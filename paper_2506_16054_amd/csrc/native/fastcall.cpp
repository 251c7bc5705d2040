// The calls that a program makes once per attention layer, from Python tensors to the C ABI without ctypes: at small layers
// the host's work is all of the time, and of the 8 us that a call took through ctypes some 5 went into attribute look-ups of
// its tensors and the conversion of its 15 to 20 arguments.
//
// A function here takes the arguments of the binding's function of the same name and either makes the call and returns
// its status, or returns None without having done anything, whenever an argument is not plainly what the call wants: another
// type, shape, layout or device, a tensor subclass or one that a transform has wrapped.  The binding then goes through its own
// checks, which raise the error or accept what this file does not know.  Nothing is kept between calls.
//
// Built as an extension module into lib/ (build.py); holds no arithmetic of the method.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <cstring>
#include <initializer_list>

#include "paro.h"

namespace {

// the library's entry points and the binding's shape type, handed over by the binding that has loaded the library
PyTypeObject* g_shape;
decltype(&paro_permute_quantize_qkv) g_qkv;
decltype(&paro_permute_quantize_qkv_keep) g_qkv_keep;
decltype(&paro_sparse_attn) g_attn;
decltype(&paro_sparse_attn_unpermuted) g_attn_unpermuted;
decltype(&paro_unpermute) g_unpermute;
decltype(&paro_mask_to_blocklist_device) g_expand;
decltype(&paro_permute_quantize_kv) g_kv;
decltype(&paro_permute_quantize_qkv_smoothed) g_qkv_smoothed;
decltype(&paro_sparse_attn_unpermuted_rawq) g_rawq;

// What follows from a shape: as the binding's _Dims.
struct Dims {
    paro_shape s;
    int64_t n, k, npad;
    bool read(PyObject* o) {
        Py_buffer b;
        if (Py_TYPE(o) != g_shape) return false;
        if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) {
            PyErr_Clear();
            return false;
        }
        const bool ok = b.len == (Py_ssize_t)sizeof(s);
        if (ok) memcpy(&s, b.buf, sizeof(s));
        PyBuffer_Release(&b);
        if (!ok || s.B < 1 || s.nh < 1 || s.d < 1 || s.F < 1 || s.Hg < 1 || s.Wg < 1 || s.T_text < 0 || s.block < 1) return false;
        n = (int64_t)s.F * s.Hg * s.Wg + s.T_text;
        k = (n + s.block - 1) / s.block;
        npad = k * s.block;
        return true;
    }
};

// A plain, contiguous tensor on the GPU.
const at::Tensor* plain(PyObject* o) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    constexpr c10::DispatchKeySet wrapped({c10::DispatchKey::Python, c10::DispatchKey::PythonTLSSnapshot, c10::DispatchKey::Functionalize,
                                           c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::FuncTorchGradWrapper,
                                           c10::DispatchKey::FuncTorchBatchedDecomposition, c10::DispatchKey::FuncTorchDynamicLayerFrontMode,
                                           c10::DispatchKey::FuncTorchDynamicLayerBackMode, c10::DispatchKey::Batched, c10::DispatchKey::Conjugate,
                                           c10::DispatchKey::Negative, c10::DispatchKey::ZeroTensor});
    if (!t.defined() || t.layout() != at::kStrided || !t.is_cuda() || t.key_set().has_any(wrapped) || !t.has_storage() || !t.is_contiguous())
        return nullptr;
    return &t;
}
const at::Tensor* of_shape(PyObject* o, std::initializer_list<int64_t> shape) {
    const at::Tensor* t = plain(o);
    return t && t->sizes().equals(c10::IntArrayRef(shape.begin(), shape.size())) ? t : nullptr;
}
const at::Tensor* typed(PyObject* o, std::initializer_list<int64_t> shape, at::ScalarType type) {
    const at::Tensor* t = of_shape(o, shape);
    return t && t->scalar_type() == type ? t : nullptr;
}
// [cap] of a type, or any shape of it
const at::Tensor* of_type(PyObject* o, at::ScalarType type) {
    const at::Tensor* t = plain(o);
    return t && t->scalar_type() == type ? t : nullptr;
}
bool dtype_of(const at::Tensor& t, paro_dtype* dtype) {
    if (t.scalar_type() == at::kFloat) *dtype = PARO_F32;
    else if (t.scalar_type() == at::kBFloat16) *dtype = PARO_BF16;
    else return false;
    return true;
}
const at::Tensor* rows_of(PyObject* o, const Dims& m, long bits) { return of_shape(o, {m.s.B, m.s.nh, m.npad, bits == 4 ? m.s.d / 2 : m.s.d}); }
const at::Tensor* vt_of(PyObject* o, const Dims& m, long bits) { return of_shape(o, {m.s.B, m.s.nh, m.k, m.s.d, bits == 4 ? m.s.block / 2 : m.s.block}); }
bool code_type(const at::Tensor* t, long bits) { return t && t->scalar_type() == (bits == 16 ? at::kBFloat16 : at::kChar); }
const at::Tensor* scales_of(PyObject* o, const Dims& m) { return typed(o, {m.s.B, m.s.nh, m.k}, at::kFloat); }

// nh order ids in a contiguous uint8 array of one dimension
struct PermIds {
    Py_buffer b;
    bool held = false;
    bool read(PyObject* o, int nh) {
        if (PyBytes_Check(o)) return false;  // numpy reads the text in it, not the bytes
        if (PyObject_GetBuffer(o, &b, PyBUF_FORMAT | PyBUF_C_CONTIGUOUS) != 0) {
            PyErr_Clear();
            return false;
        }
        held = true;
        return b.ndim == 1 && b.itemsize == 1 && b.shape[0] == nh && b.format && b.format[0] == 'B' && b.format[1] == 0;
    }
    const uint8_t* data() const { return (const uint8_t*)b.buf; }
    ~PermIds() {
        if (held) PyBuffer_Release(&b);
    }
};

// a plain int (a bool or another integer type goes the binding's way)
bool number(PyObject* o, long* v) {
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    *v = PyLong_AsLongAndOverflow(o, &overflow);
    return overflow == 0 && *v >= -0x7fffffffL && *v <= 0x7fffffffL;
}
void* stream() { return (void*)c10::hip::getCurrentHIPStream().stream(); }
void* ptr(const at::Tensor* t) { return t->data_ptr(); }

// C++ exceptions (a tensor whose storage refuses, a device that is gone) must not cross into the interpreter.
template <typename F>
PyObject* guarded(F&& f) {
    try {
        return f();
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}
#define PARO_DECLINE Py_RETURN_NONE

// s, bits_qk, bits_pv, perm_ids, the inputs from tensor `first` (0 q, 1 k) on, ..., and from argument `at` on their codes and scales in turn
struct QkvArgs {
    Dims m;
    long qk, pv;
    PermIds ids;
    int first;
    const at::Tensor *in[3], *codes[3], *scales[3];
    paro_dtype dtype;
    void *p[3], *c[3], *st;
    float* f[3];
    bool read(PyObject* const* a, int from, int at) {
        first = from;
        if (!m.read(a[0]) || !number(a[1], &qk) || !number(a[2], &pv) || !ids.read(a[3], m.s.nh)) return false;
        for (int i = first; i < 3; ++i) {
            in[i] = of_shape(a[4 + i - first], {m.s.B, m.s.nh, m.n, m.s.d});
            if (!in[i] || in[i]->scalar_type() != in[first]->scalar_type()) return false;
        }
        if (!dtype_of(*in[first], &dtype)) return false;
        for (int i = first; i < 3; ++i) {
            const long bits = i == 2 ? pv : qk;
            PyObject* const* pair = a + at + 2 * (i - first);
            codes[i] = i == 2 ? vt_of(pair[0], m, bits) : rows_of(pair[0], m, bits);
            scales[i] = scales_of(pair[1], m);
            if (!code_type(codes[i], bits) || !scales[i]) return false;
        }
        return true;
    }
    void pointers() {
        st = stream();
        for (int i = first; i < 3; ++i) {
            p[i] = ptr(in[i]);
            c[i] = ptr(codes[i]);
            f[i] = (float*)ptr(scales[i]);
        }
    }
};

PyObject* quantize_qkv(PyObject* const* a, Py_ssize_t count, bool keep) {
    // s, bits_qk, bits_pv, perm_ids, q, k, v, [qp, kp, vp,] q_codes, sq, k_codes, sk, v_codes, sv
    if (count != (keep ? 16 : 13) || !g_shape) PARO_DECLINE;
    QkvArgs x;
    if (!x.read(a, 0, keep ? 10 : 7)) PARO_DECLINE;
    const at::Tensor* kept[3] = {nullptr, nullptr, nullptr};
    for (int i = 0; keep && i < 3; ++i)
        if (!(kept[i] = typed(a[7 + i], {x.m.s.B, x.m.s.nh, x.m.npad, x.m.s.d}, x.in[0]->scalar_type()))) PARO_DECLINE;
    void* r[3];
    for (int i = 0; i < 3; ++i) r[i] = keep ? ptr(kept[i]) : nullptr;
    x.pointers();
    int status;
    Py_BEGIN_ALLOW_THREADS;
    status = keep ? g_qkv_keep(&x.m.s, x.dtype, (int)x.qk, (int)x.pv, x.ids.data(), x.p[0], x.p[1], x.p[2], r[0], r[1], r[2], x.c[0], x.f[0], x.c[1],
                               x.f[1], x.c[2], x.f[2], x.st)
                  : g_qkv(&x.m.s, x.dtype, (int)x.qk, (int)x.pv, x.ids.data(), x.p[0], x.p[1], x.p[2], x.c[0], x.f[0], x.c[1], x.f[1], x.c[2], x.f[2],
                          x.st);
    Py_END_ALLOW_THREADS;
    return PyLong_FromLong(status);
}

PyObject* quantize_kv(PyObject* const* a, Py_ssize_t count) {  // s, bits_qk, bits_pv, perm_ids, k, v, k_codes, sk, v_codes, sv
    if (count != 10 || !g_shape) PARO_DECLINE;
    QkvArgs x;
    if (!x.read(a, 1, 6)) PARO_DECLINE;
    x.pointers();
    int status;
    Py_BEGIN_ALLOW_THREADS;
    status = g_kv(&x.m.s, x.dtype, (int)x.qk, (int)x.pv, x.ids.data(), x.p[1], x.p[2], x.c[1], x.f[1], x.c[2], x.f[2], x.st);
    Py_END_ALLOW_THREADS;
    return PyLong_FromLong(status);
}

PyObject* quantize_qkv_smoothed(PyObject* const* a, Py_ssize_t count) {
    // s, bits_qk, bits_pv, perm_ids, q, k, v, k_mean, q_codes, sq, k_codes, sk, v_codes, sv
    if (count != 14 || !g_shape) PARO_DECLINE;
    QkvArgs x;
    if (!x.read(a, 0, 8)) PARO_DECLINE;
    const at::Tensor* mean = typed(a[7], {x.m.s.B, x.m.s.nh, x.m.s.d}, at::kFloat);
    if (!mean) PARO_DECLINE;
    float* mp = (float*)ptr(mean);
    x.pointers();
    int status;
    Py_BEGIN_ALLOW_THREADS;
    status = g_qkv_smoothed(&x.m.s, x.dtype, (int)x.qk, (int)x.pv, x.ids.data(), x.p[0], x.p[1], x.p[2], mp, x.c[0], x.f[0], x.c[1], x.f[1], x.c[2],
                            x.f[2], x.st);
    Py_END_ALLOW_THREADS;
    return PyLong_FromLong(status);
}

PyObject* attention(PyObject* const* a, Py_ssize_t count, bool unpermuted) {
    // s, bits_qk, bits_pv, q, sq, k, sk, v, sv, row_ptr, col_idx, [perm_ids,] o, row_order
    if (count != (unpermuted ? 14 : 13) || !g_shape) PARO_DECLINE;
    Dims m;
    long qk, pv;
    PermIds ids;
    if (!m.read(a[0]) || !number(a[1], &qk) || !number(a[2], &pv)) PARO_DECLINE;
    const at::Tensor* q = rows_of(a[3], m, qk);
    const at::Tensor* k = rows_of(a[5], m, qk);
    const at::Tensor* v = vt_of(a[7], m, pv);
    if (!q || !k || !v) PARO_DECLINE;
    const at::Tensor* scales[3];
    for (int i = 0; i < 3; ++i) {
        scales[i] = a[4 + 2 * i] == Py_None ? nullptr : scales_of(a[4 + 2 * i], m);
        if (!scales[i] && a[4 + 2 * i] != Py_None) PARO_DECLINE;
    }
    const at::Tensor* row_ptr = typed(a[9], {m.s.nh, m.k + 1}, at::kInt);
    const at::Tensor* cols = of_type(a[10], at::kInt);
    if (!row_ptr || !cols) PARO_DECLINE;
    if (unpermuted && !ids.read(a[11], m.s.nh)) PARO_DECLINE;
    PyObject* const* tail = a + (unpermuted ? 12 : 11);
    const at::Tensor* o = of_shape(tail[0], {m.s.B, m.s.nh, unpermuted ? m.n : m.npad, m.s.d});
    paro_dtype dtype;
    if (!o || !dtype_of(*o, &dtype)) PARO_DECLINE;
    const at::Tensor* order = nullptr;
    if (tail[1] != Py_None && !(order = typed(tail[1], {(int64_t)m.s.B * m.s.nh * m.k}, at::kInt))) PARO_DECLINE;
    void* st = stream();
    const int64_t nnz = cols->numel();
    float* f[3];
    for (int i = 0; i < 3; ++i) f[i] = scales[i] ? (float*)ptr(scales[i]) : nullptr;
    void *qp = ptr(q), *kp = ptr(k), *vp = ptr(v), *op = ptr(o);
    const int32_t* rp = (const int32_t*)ptr(row_ptr);
    const int32_t* ci = nnz ? (const int32_t*)ptr(cols) : nullptr;
    const int32_t* ro = order ? (const int32_t*)ptr(order) : nullptr;
    int status;
    Py_BEGIN_ALLOW_THREADS;
    status = unpermuted
        ? g_attn_unpermuted(&m.s, (int)qk, (int)pv, qp, f[0], kp, f[1], vp, f[2], rp, ci, nnz, ro, ids.data(), dtype, op, st)
        : g_attn(&m.s, (int)qk, (int)pv, qp, f[0], kp, f[1], vp, f[2], rp, ci, nnz, ro, dtype, op, st);
    Py_END_ALLOW_THREADS;
    return PyLong_FromLong(status);
}

PyObject* attention_rawq(PyObject* const* a, Py_ssize_t count) {  // s, bits_pv, q, k, sk, v, sv, row_ptr, col_idx, perm_ids, o, row_order
    if (count != 12 || !g_shape) PARO_DECLINE;
    Dims m;
    long pv;
    PermIds ids;
    if (!m.read(a[0]) || !number(a[1], &pv) || !ids.read(a[9], m.s.nh)) PARO_DECLINE;
    const at::Tensor* q = of_shape(a[2], {m.s.B, m.s.nh, m.n, m.s.d});
    const at::Tensor* k = rows_of(a[3], m, 8);
    const at::Tensor* v = vt_of(a[5], m, pv);
    const at::Tensor *sk = scales_of(a[4], m), *sv = scales_of(a[6], m);
    paro_dtype q_dtype, dtype;
    if (!q || !dtype_of(*q, &q_dtype) || !k || k->scalar_type() != at::kChar || !v || v->scalar_type() != at::kChar || !sk || !sv) PARO_DECLINE;
    const at::Tensor* row_ptr = typed(a[7], {m.s.nh, m.k + 1}, at::kInt);
    const at::Tensor* cols = of_type(a[8], at::kInt);
    const at::Tensor* o = of_shape(a[10], {m.s.B, m.s.nh, m.n, m.s.d});
    if (!row_ptr || !cols || !o || !dtype_of(*o, &dtype)) PARO_DECLINE;
    const at::Tensor* order = nullptr;
    if (a[11] != Py_None && !(order = typed(a[11], {(int64_t)m.s.B * m.s.nh * m.k}, at::kInt))) PARO_DECLINE;
    void* st = stream();
    const int64_t nnz = cols->numel();
    void *qp = ptr(q), *kp = ptr(k), *vp = ptr(v), *op = ptr(o);
    const float *skp = (const float*)ptr(sk), *svp = (const float*)ptr(sv);
    const int32_t* rp = (const int32_t*)ptr(row_ptr);
    const int32_t* ci = nnz ? (const int32_t*)ptr(cols) : nullptr;
    const int32_t* ro = order ? (const int32_t*)ptr(order) : nullptr;
    int status;
    Py_BEGIN_ALLOW_THREADS;
    status = g_rawq(&m.s, q_dtype, (int)pv, qp, kp, skp, vp, svp, rp, ci, nnz, ro, ids.data(), dtype, op, st);
    Py_END_ALLOW_THREADS;
    return PyLong_FromLong(status);
}

PyObject* inverse_reorder(PyObject* const* a, Py_ssize_t count) {  // s, perm_ids, op, o
    if (count != 4 || !g_shape) PARO_DECLINE;
    Dims m;
    PermIds ids;
    if (!m.read(a[0]) || !ids.read(a[1], m.s.nh)) PARO_DECLINE;
    const at::Tensor* op = of_shape(a[2], {m.s.B, m.s.nh, m.npad, m.s.d});
    paro_dtype dtype;
    if (!op || !dtype_of(*op, &dtype)) PARO_DECLINE;
    const at::Tensor* o = typed(a[3], {m.s.B, m.s.nh, m.n, m.s.d}, op->scalar_type());
    if (!o) PARO_DECLINE;
    void *st = stream(), *src = ptr(op), *dst = ptr(o);
    int status;
    Py_BEGIN_ALLOW_THREADS;
    status = g_unpermute(&m.s, dtype, ids.data(), src, dst, st);
    Py_END_ALLOW_THREADS;
    return PyLong_FromLong(status);
}

PyObject* expand(PyObject* const* a, Py_ssize_t count) {  // nh, k, bitmask, row_ptr, col_idx or None, nnz or None
    if (count != 6 || !g_shape) PARO_DECLINE;
    long nh, k;
    if (!number(a[0], &nh) || !number(a[1], &k) || nh < 1 || k < 1) PARO_DECLINE;
    const at::Tensor* bits = typed(a[2], {nh, (k * k + 7) / 8}, at::kByte);
    const at::Tensor* row_ptr = typed(a[3], {nh, k + 1}, at::kInt);
    const at::Tensor* cols = a[4] == Py_None ? nullptr : of_type(a[4], at::kInt);
    const at::Tensor* nnz = a[5] == Py_None ? nullptr : typed(a[5], {1}, at::kInt);
    if (!bits || !row_ptr || (!cols && a[4] != Py_None) || (!nnz && a[5] != Py_None)) PARO_DECLINE;
    const int64_t cap = cols ? cols->numel() : 0;
    void* st = stream();
    const uint8_t* bm = (const uint8_t*)ptr(bits);
    int32_t *rp = (int32_t*)ptr(row_ptr), *ci = cap ? (int32_t*)ptr(cols) : nullptr, *nz = nnz ? (int32_t*)ptr(nnz) : nullptr;
    int status;
    Py_BEGIN_ALLOW_THREADS;
    status = g_expand((int)nh, (int)k, bm, rp, ci, cap, nz, st);
    Py_END_ALLOW_THREADS;
    return PyLong_FromLong(status);
}

PyObject* f_qkv(PyObject*, PyObject* const* a, Py_ssize_t n) { return guarded([&] { return quantize_qkv(a, n, false); }); }
PyObject* f_qkv_keep(PyObject*, PyObject* const* a, Py_ssize_t n) { return guarded([&] { return quantize_qkv(a, n, true); }); }
PyObject* f_attn(PyObject*, PyObject* const* a, Py_ssize_t n) { return guarded([&] { return attention(a, n, false); }); }
PyObject* f_attn_unpermuted(PyObject*, PyObject* const* a, Py_ssize_t n) { return guarded([&] { return attention(a, n, true); }); }
PyObject* f_unpermute(PyObject*, PyObject* const* a, Py_ssize_t n) { return guarded([&] { return inverse_reorder(a, n); }); }
PyObject* f_kv(PyObject*, PyObject* const* a, Py_ssize_t n) { return guarded([&] { return quantize_kv(a, n); }); }
PyObject* f_qkv_smoothed(PyObject*, PyObject* const* a, Py_ssize_t n) { return guarded([&] { return quantize_qkv_smoothed(a, n); }); }
PyObject* f_rawq(PyObject*, PyObject* const* a, Py_ssize_t n) { return guarded([&] { return attention_rawq(a, n); }); }
PyObject* f_expand(PyObject*, PyObject* const* a, Py_ssize_t n) { return guarded([&] { return expand(a, n); }); }

PyObject* f_bind(PyObject*, PyObject* args) {  // the shape type, then the addresses in the order of the declarations above
    PyObject* shape;
    unsigned long long p[9];
    if (!PyArg_ParseTuple(args, "O!KKKKKKKKK", &PyType_Type, &shape, p, p + 1, p + 2, p + 3, p + 4, p + 5, p + 6, p + 7, p + 8)) return nullptr;
    Py_INCREF(shape);  // for the life of the process, like the library
    g_shape = (PyTypeObject*)shape;
    g_qkv = (decltype(g_qkv))(uintptr_t)p[0];
    g_qkv_keep = (decltype(g_qkv_keep))(uintptr_t)p[1];
    g_attn = (decltype(g_attn))(uintptr_t)p[2];
    g_attn_unpermuted = (decltype(g_attn_unpermuted))(uintptr_t)p[3];
    g_unpermute = (decltype(g_unpermute))(uintptr_t)p[4];
    g_expand = (decltype(g_expand))(uintptr_t)p[5];
    g_kv = (decltype(g_kv))(uintptr_t)p[6];
    g_qkv_smoothed = (decltype(g_qkv_smoothed))(uintptr_t)p[7];
    g_rawq = (decltype(g_rawq))(uintptr_t)p[8];
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", f_bind, METH_VARARGS, nullptr},
    {"paro_permute_quantize_qkv", (PyCFunction)(void (*)(void))f_qkv, METH_FASTCALL, nullptr},
    {"paro_permute_quantize_qkv_keep", (PyCFunction)(void (*)(void))f_qkv_keep, METH_FASTCALL, nullptr},
    {"paro_sparse_attn", (PyCFunction)(void (*)(void))f_attn, METH_FASTCALL, nullptr},
    {"paro_sparse_attn_unpermuted", (PyCFunction)(void (*)(void))f_attn_unpermuted, METH_FASTCALL, nullptr},
    {"paro_unpermute", (PyCFunction)(void (*)(void))f_unpermute, METH_FASTCALL, nullptr},
    {"paro_mask_to_blocklist_device", (PyCFunction)(void (*)(void))f_expand, METH_FASTCALL, nullptr},
    {"paro_permute_quantize_kv", (PyCFunction)(void (*)(void))f_kv, METH_FASTCALL, nullptr},
    {"paro_permute_quantize_qkv_smoothed", (PyCFunction)(void (*)(void))f_qkv_smoothed, METH_FASTCALL, nullptr},
    {"paro_sparse_attn_unpermuted_rawq", (PyCFunction)(void (*)(void))f_rawq, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "paro_fastcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_paro_fastcall(void) {
    PyObject* m = PyModule_Create(&module);
    // the torch whose tensors this file knows the layout of; the binding loads it beside no other
    if (m && PyModule_AddStringConstant(m, "built_for", PARO_TORCH_VERSION) != 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
