// The calls of the binding for the ordinary case: every argument as the entry points want it, tensors in GPU memory. Anything
// else (NOT_HANDLED) goes through binding.py, which checks again, converts what can be converted and names what cannot be.
//
// The last argument of each is the binding's `stream`, passes and axes are what its caller gave.
// Why: a small kernel lasts 3 .. 5 us and HIP takes 2.9 us to launch it, while the checks in Python (a dozen attributes of five
// or six tensors) took 2.3 .. 3 us and the call through ctypes 0.6 us. Here the checks cost 0.1 us and the call 0.2 us.
// The library's entry points are handed over by address, so that this module and the binding call the same library.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

namespace {

constexpr long NOT_HANDLED = -1;
constexpr int kRowwise = 1, kColwise = 2, kTiled = 1;
// entry points, in the order of the names below
enum { QUANTIZE, GEMM, GEMM_MODE, DEQUANTIZE, GEMM_BF16, GEMM_QUANTIZE, FP4_QUANTIZE, FP4_GEMM, FP6_QUANTIZE, ENTRY_POINTS };
const char *const kNames[ENTRY_POINTS] = {"mxfp8_quantize_mode_ex", "mxfp8_gemm_ex", "mxfp8_gemm_mode_ex", "mxfp8_dequantize_mode_ex",
                                          "mxfp8_gemm_bf16", "mxfp8_gemm_quantize_ex", "mxfp8_fp4_quantize_ex",
                                          "mxfp8_fp4_gemm_ex", "mxfp8_fp6_quantize_ex"};
void *entry[ENTRY_POINTS];
// The binding's own: names and constants of passes and axes (dicts), and the function that turns its `stream` argument into a handle.
PyObject *passes, *axes, *stream_handle;

// Arguments of a call, taken one after the other; `ok` turns false at the first one that is not what it has to be.
struct Args {
    PyObject *const *args;
    Py_ssize_t left;
    bool ok = true;
    PyObject *next()
    {
        if (left <= 0) {
            ok = false;
            return Py_None;
        }
        --left;
        return *args++;
    }
    int64_t number(int64_t lo, int64_t hi)
    {
        PyObject *o = next();
        if (!PyLong_CheckExact(o)) {
            ok = false;
            return lo;
        }
        int overflow = 0;
        const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
        if (overflow || v < lo || v > hi)
            ok = false;
        return v;
    }
    // what `table` has for the next argument
    int64_t code(PyObject *table, int64_t lo, int64_t hi)
    {
        PyObject *v = table ? PyDict_GetItem(table, next()) : nullptr;  // (nullptr also for what cannot be looked up)
        const long long c = v && PyLong_CheckExact(v) ? PyLong_AsLong(v) : lo - 1;
        if (c < lo || c > hi)
            ok = false;
        return c;
    }
    // a tensor in GPU memory; nullptr for None where that is allowed
    const at::Tensor *tensor(bool none_allowed = false)
    {
        PyObject *o = next();
        if (o == Py_None && none_allowed)
            return nullptr;
        if (THPVariable_CheckTypeExact(Py_TYPE(o))) {  // subclasses may answer for themselves
            const at::Tensor &t = THPVariable_Unpack(o);
            if (t.defined() && t.layout() == at::kStrided && t.is_cuda())
                return &t;
        }
        ok = false;
        return nullptr;
    }
};

uint8_t *ptr(const at::Tensor *t) { return t ? static_cast<uint8_t *>(t->data_ptr()) : nullptr; }
bool dense_bytes(const at::Tensor &t) { return t.scalar_type() == at::kByte && t.is_contiguous(); }
bool dense_matrix(const at::Tensor &t, int64_t rows, int64_t cols) { return t.dim() == 2 && t.size(0) == rows && t.size(1) == cols && dense_bytes(t); }
// scale bytes of an operand [rows x cols]
bool scales(const at::Tensor &s, int64_t rows, int64_t cols, int64_t layout)
{
    if (!dense_bytes(s) || cols % 32)
        return false;
    if (layout == kTiled)
        return s.numel() >= (rows + 63) / 64 * ((cols / 32 + 3) / 4) * 256;
    return s.dim() == 2 && s.size(0) == rows && s.size(1) == cols / 32;
}
// a matrix of FP32 or BF16 values with contiguous rows
struct Values {
    bool ok;
    int dtype;
    int64_t ld;
};
Values values(const at::Tensor &t, int64_t rows, int64_t cols)
{
    const auto type = t.scalar_type();
    const bool ok = t.dim() == 2 && t.size(0) == rows && t.size(1) == cols && rows > 0 && cols > 0 && t.stride(1) == 1 &&
                    (type == at::kFloat || type == at::kBFloat16);
    return {ok, type == at::kBFloat16 ? 1 : 0, ok && rows > 1 ? t.stride(0) : cols};
}

PyObject *not_handled() { return PyLong_FromLong(NOT_HANDLED); }
// The binding asks for the stream after its checks, so that a wrong tensor is reported as one on a machine without a GPU too.
template <class F, class... A> PyObject *call(int which, PyObject *stream, A... args)
{
    if (!entry[which] || !stream_handle)
        return not_handled();
    PyObject *h = PyObject_CallFunctionObjArgs(stream_handle, stream, nullptr);
    if (!h)
        return nullptr;
    void *handle = PyLong_CheckExact(h) ? PyLong_AsVoidPtr(h) : nullptr;
    const bool ok = PyLong_CheckExact(h) && !PyErr_Occurred();
    Py_DECREF(h);
    if (!ok) {
        PyErr_Clear();
        return not_handled();
    }
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = reinterpret_cast<F>(entry[which])(args..., handle);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// The copies of a quantizer: q_row, s_row, q_colT, s_colT; `num` / `den` bytes per element
struct Copies {
    const at::Tensor *q_row, *s_row, *q_colT, *s_colT;
};
bool copies(Args &a, Copies &c, int64_t rows, int64_t cols, int64_t axis, int64_t layout, int num, int den)
{
    const bool row = axis & kRowwise, col = axis & kColwise;
    return a.ok && (!row || (c.q_row && c.s_row && dense_bytes(*c.q_row) && c.q_row->numel() == rows * cols / den * num && scales(*c.s_row, rows, cols, layout))) &&
           (!col || (c.q_colT && c.s_colT && dense_bytes(*c.q_colT) && c.q_colT->numel() == rows * cols / den * num && scales(*c.s_colT, cols, rows, layout)));
}

using I = int64_t;
using P = const uint8_t *;
using Q = uint8_t *;

// src, axis, element, rule, q_row, s_row, q_colT, s_colT, layout, stream; FP4: no element and rule, FP6: no rule
template <int WHICH> PyObject *quantize(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    Args a{args, n};
    const at::Tensor *src = a.tensor();
    const int64_t axis = a.code(axes, 1, 3), element = WHICH == FP4_QUANTIZE ? 0 : a.number(0, 1), rule = WHICH == QUANTIZE ? a.number(0, 1) : 0;
    Copies c;
    c.q_row = a.tensor(true);
    c.s_row = a.tensor(true);
    c.q_colT = a.tensor(true);
    c.s_colT = a.tensor(true);
    const int64_t layout = a.number(0, 1);
    PyObject *stream = a.next();
    if (!a.ok || a.left || src->dim() != 2)
        return not_handled();
    const int64_t rows = src->size(0), cols = src->size(1);
    const Values v = values(*src, rows, cols);
    if (!v.ok || !copies(a, c, rows, cols, axis, layout, WHICH == FP6_QUANTIZE ? 3 : 1, WHICH == FP6_QUANTIZE ? 4 : WHICH == FP4_QUANTIZE ? 2 : 1))
        return not_handled();
    if constexpr (WHICH == QUANTIZE)
        return call<int (*)(P, int, I, I, I, int, int, int, Q, Q, Q, Q, int, void *)>(
            WHICH, stream, ptr(src), v.dtype, rows, cols, v.ld, (int)axis, (int)element, (int)rule, ptr(c.q_row), ptr(c.s_row), ptr(c.q_colT),
            ptr(c.s_colT), (int)layout);
    else if constexpr (WHICH == FP6_QUANTIZE)
        return call<int (*)(P, int, I, I, I, int, int, Q, Q, Q, Q, int, void *)>(WHICH, stream, ptr(src), v.dtype, rows, cols, v.ld, (int)axis, (int)element,
                                                                                ptr(c.q_row), ptr(c.s_row), ptr(c.q_colT), ptr(c.s_colT), (int)layout);
    else
        return call<int (*)(P, int, I, I, I, int, Q, Q, Q, Q, int, void *)>(WHICH, stream, ptr(src), v.dtype, rows, cols, v.ld, (int)axis, ptr(c.q_row),
                                                                           ptr(c.s_row), ptr(c.q_colT), ptr(c.s_colT), (int)layout);
}

// pass, a_q, a_s, [a_element,] b_q, b_s, [b_element,] c, layout, max_workgroups, stream
template <int WHICH> PyObject *gemm(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    Args a{args, n};
    const int64_t pass = a.code(passes, 0, 2);
    const at::Tensor *a_q = a.tensor(), *a_s = a.tensor();
    const int64_t a_element = WHICH == GEMM_MODE ? a.number(0, 1) : 0;
    const at::Tensor *b_q = a.tensor(), *b_s = a.tensor();
    const int64_t b_element = WHICH == GEMM_MODE ? a.number(0, 1) : 0;
    const at::Tensor *c = a.tensor();
    const int64_t layout = a.number(0, 1), bound = a.number(0, INT32_MAX);
    PyObject *stream = a.next();
    if (!a.ok || a.left || a_q->dim() != 2 || b_q->dim() != 2)
        return not_handled();
    const int64_t M = a_q->size(0), N = b_q->size(0), bytes = a_q->size(1), K = WHICH == FP4_GEMM ? 2 * bytes : bytes;
    const Values v = values(*c, M, N);
    if (!v.ok || !dense_matrix(*a_q, M, bytes) || !dense_matrix(*b_q, N, bytes) || !scales(*a_s, M, K, layout) || !scales(*b_s, N, K, layout))
        return not_handled();
    if constexpr (WHICH == GEMM_MODE)
        return call<int (*)(int, P, P, int, P, P, int, I, I, I, void *, int, I, int, int32_t, void *)>(
            WHICH, stream, (int)pass, ptr(a_q), ptr(a_s), (int)a_element, ptr(b_q), ptr(b_s), (int)b_element, M, N, K, (void *)ptr(c), v.dtype, v.ld,
            (int)layout, (int32_t)bound);
    else
        return call<int (*)(int, P, P, P, P, I, I, I, void *, int, I, int, int32_t, void *)>(
            WHICH, stream, (int)pass, ptr(a_q), ptr(a_s), ptr(b_q), ptr(b_s), M, N, K, (void *)ptr(c), v.dtype, v.ld, (int)layout, (int32_t)bound);
}

// q, s, element, dst, layout, stream
PyObject *dequantize(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    Args a{args, n};
    const at::Tensor *q = a.tensor(), *s = a.tensor();
    const int64_t element = a.number(0, 1);
    const at::Tensor *dst = a.tensor();
    const int64_t layout = a.number(0, 1);
    PyObject *stream = a.next();
    if (!a.ok || a.left || q->dim() != 2)
        return not_handled();
    const int64_t rows = q->size(0), cols = q->size(1);
    const Values v = values(*dst, rows, cols);
    if (!v.ok || !dense_bytes(*q) || !scales(*s, rows, cols, layout))
        return not_handled();
    return call<int (*)(P, P, I, I, int, void *, int, I, int, void *)>(DEQUANTIZE, stream, ptr(q), ptr(s), rows, cols, (int)element, (void *)ptr(dst), v.dtype, v.ld,
                                                                      (int)layout);
}

// a, b, c, max_workgroups, stream
PyObject *gemm_bf16(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    Args a{args, n};
    const at::Tensor *x = a.tensor(), *y = a.tensor(), *c = a.tensor();
    const int64_t bound = a.number(0, INT32_MAX);
    PyObject *stream = a.next();
    if (!a.ok || a.left || x->dim() != 2 || y->dim() != 2)
        return not_handled();
    const int64_t M = x->size(0), N = y->size(0), K = x->size(1);
    const Values v = values(*c, M, N);
    if (!v.ok || y->size(1) != K || x->scalar_type() != at::kBFloat16 || y->scalar_type() != at::kBFloat16 || !x->is_contiguous() || !y->is_contiguous())
        return not_handled();
    return call<int (*)(P, P, I, I, I, void *, int, I, int32_t, void *)>(GEMM_BF16, stream, ptr(x), ptr(y), M, N, K, (void *)ptr(c), v.dtype, v.ld, (int32_t)bound);
}

// pass, a_q, a_s, b_q, b_s, c, axis, cq_row, cs_row, cq_colT, cs_colT, layout, max_workgroups, stream
PyObject *gemm_quantize(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    Args a{args, n};
    const int64_t pass = a.code(passes, 0, 2);
    const at::Tensor *a_q = a.tensor(), *a_s = a.tensor(), *b_q = a.tensor(), *b_s = a.tensor(), *c = a.tensor();
    const int64_t axis = a.code(axes, 1, 3);
    Copies q;
    q.q_row = a.tensor(true);
    q.s_row = a.tensor(true);
    q.q_colT = a.tensor(true);
    q.s_colT = a.tensor(true);
    const int64_t layout = a.number(0, 1), bound = a.number(0, INT32_MAX);
    PyObject *stream = a.next();
    if (!a.ok || a.left || a_q->dim() != 2 || b_q->dim() != 2)
        return not_handled();
    const int64_t M = a_q->size(0), N = b_q->size(0), K = a_q->size(1);
    const Values v = values(*c, M, N);
    if (!v.ok || v.dtype != 1 || !dense_matrix(*a_q, M, K) || !dense_matrix(*b_q, N, K) || !scales(*a_s, M, K, layout) || !scales(*b_s, N, K, layout) ||
        !copies(a, q, M, N, axis, layout, 1, 1) || ((axis & kRowwise) && !dense_matrix(*q.q_row, M, N)) || ((axis & kColwise) && !dense_matrix(*q.q_colT, N, M)))
        return not_handled();
    return call<int (*)(int, P, P, P, P, I, I, I, void *, I, int, Q, Q, Q, Q, int, int32_t, void *)>(
        GEMM_QUANTIZE, stream, (int)pass, ptr(a_q), ptr(a_s), ptr(b_q), ptr(b_s), M, N, K, (void *)ptr(c), v.ld, (int)axis, ptr(q.q_row), ptr(q.s_row),
        ptr(q.q_colT), ptr(q.s_colT), (int)layout, (int32_t)bound);
}

// {name: address} of the entry points, and the binding's "passes", "axes" and "stream"
PyObject *bind(PyObject *, PyObject *table)
{
    if (!PyDict_Check(table)) {
        PyErr_SetString(PyExc_TypeError, "bind() takes a dict of addresses");
        return nullptr;
    }
    const struct {
        const char *name;
        PyObject **to;
        bool dict;
    } own[] = {{"passes", &passes, true}, {"axes", &axes, true}, {"stream", &stream_handle, false}};
    for (const auto &o : own) {
        PyObject *v = PyDict_GetItemString(table, o.name);
        if (v && (o.dict ? !PyDict_Check(v) : !PyCallable_Check(v))) {
            PyErr_Format(PyExc_TypeError, "bind(): bad \"%s\"", o.name);
            return nullptr;
        }
        Py_XINCREF(v);
        Py_XSETREF(*o.to, v);
    }
    for (int i = 0; i < ENTRY_POINTS; ++i) {
        PyObject *v = PyDict_GetItemString(table, kNames[i]);
        entry[i] = v ? PyLong_AsVoidPtr(v) : nullptr;
        if (PyErr_Occurred())
            return nullptr;
    }
    Py_RETURN_NONE;
}

// Tensors without memory of their own (traced, batched) throw when they are asked for it: the binding's checks say so.
template <PyObject *(*FN)(PyObject *, PyObject *const *, Py_ssize_t)> PyObject *guarded(PyObject *self, PyObject *const *args, Py_ssize_t n)
{
    try {
        return FN(self, args, n);
    } catch (...) {
        return not_handled();
    }
}

#define FAST(name, ...) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&guarded<__VA_ARGS__>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST("quantize", quantize<QUANTIZE>), FAST("fp4_quantize", quantize<FP4_QUANTIZE>), FAST("fp6_quantize", quantize<FP6_QUANTIZE>),
                         FAST("gemm", gemm<GEMM>), FAST("gemm_mode", gemm<GEMM_MODE>), FAST("fp4_gemm", gemm<FP4_GEMM>), FAST("dequantize", dequantize),
                         FAST("gemm_bf16", gemm_bf16), FAST("gemm_quantize", gemm_quantize), {"bind", bind, METH_O, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall(void) { return PyModule_Create(&module); }
