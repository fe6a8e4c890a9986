// Python entry points of the device functions: argument checks, output allocation and the call of the C ABI
// (include/qnn.h), as a CPython extension on torch's C++ tensors.
//
// A layer of a small network runs for 4-6 us on the GPU; through ctypes and Python-level checks each call
// took 13.5 us of host time, so that a batch-1 network was bound by the interpreter (366 us for 27 calls).
// Here a call unpacks the tensors directly (no attribute look-ups), takes the output from torch's
// allocator without the dispatcher and launches: see the figures in the design notes.
//
// Functions take positional arguments only, in the order of their Python wrappers in binding.py, which
// hold the names, defaults and documentation.  A call on tensors of the wrong kind raises TypeError or
// ValueError as before; a status other than QNN_OK goes through the `check` callable that binding.py sets.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/hip/EmptyTensor.h>
#include <c10/hip/HIPStream.h>
#include <c10/util/Exception.h>
#include <c10/util/SmallVector.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/qnn.h"

namespace {

struct PythonErrorSet {}; // thrown when a Python exception is already set

PyObject *g_check = nullptr; // binding._check(name, status): raises for a status other than QNN_OK

// names of the dictionary that qadd_params() returns
enum { P_LEFT, P_MULT_A, P_SHIFT_A, P_MULT_B, P_SHIFT_B, P_MULT_O, P_SHIFT_O, P_COUNT };
const char *const kParamNames[P_COUNT] = {"left_shift", "mult_a", "shift_a", "mult_b", "shift_b", "mult_o", "shift_o"};
PyObject *g_param_names[P_COUNT];

[[noreturn]] void type_error(const char *name, const char *what)
{
    PyErr_Format(PyExc_TypeError, "%s: expected %s", name, what);
    throw PythonErrorSet{};
}

[[noreturn]] void shape_error(const char *name, at::IntArrayRef got, at::IntArrayRef want)
{
    auto text = [](at::IntArrayRef s) {
        std::string t = "(";
        for (size_t i = 0; i < s.size(); ++i) t += (i ? ", " : "") + std::to_string(s[i]);
        return t + ")";
    };
    PyErr_Format(PyExc_ValueError, "%s has shape %s, expected %s", name, text(got).c_str(), text(want).c_str());
    throw PythonErrorSet{};
}

int64_t integer(PyObject *o)
{
    // wraps modulo 2^64 like a C integer argument; accepts what has an index, rejects floats
    const int64_t v = (int64_t)PyLong_AsUnsignedLongLongMask(o);
    if (v == -1 && PyErr_Occurred()) throw PythonErrorSet{};
    return v;
}
int32_t i32(PyObject *o) { return (int32_t)integer(o); }

// what Python's int() takes: floats are truncated
int32_t whole(PyObject *o)
{
    if (PyLong_Check(o)) return i32(o);
    PyObject *const v = PyNumber_Long(o);
    if (!v) throw PythonErrorSet{};
    const int64_t r = (int64_t)PyLong_AsUnsignedLongLongMask(v);
    Py_DECREF(v);
    return (int32_t)r;
}

float real(PyObject *o)
{
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) throw PythonErrorSet{};
    return (float)v;
}

struct Pair {
    int h, w;
};
Pair pair(PyObject *o)
{
    if (PyTuple_Check(o) && PyTuple_GET_SIZE(o) >= 2) return {i32(PyTuple_GET_ITEM(o, 0)), i32(PyTuple_GET_ITEM(o, 1))};
    Pair p;
    int *const dst[2] = {&p.h, &p.w};
    for (int i = 0; i < 2; ++i) {
        PyObject *item = PySequence_GetItem(o, i);
        if (!item) throw PythonErrorSet{};
        const int64_t v = (int64_t)PyLong_AsUnsignedLongLongMask(item);
        Py_DECREF(item);
        if (v == -1 && PyErr_Occurred()) throw PythonErrorSet{};
        *dst[i] = (int)v;
    }
    return p;
}

const at::Tensor &tensor(PyObject *o, const char *name)
{
    if (!THPVariable_Check(o)) type_error(name, "a device tensor");
    return THPVariable_Unpack(o);
}

const char *type_name(at::ScalarType t)
{
    switch (t) {
    case at::kByte: return "a contiguous device tensor of torch.uint8";
    case at::kChar: return "a contiguous device tensor of torch.int8";
    case at::kInt: return "a contiguous device tensor of torch.int32";
    case at::kFloat: return "a contiguous device tensor of torch.float32";
    default: return "a contiguous device tensor of torch.uint16";
    }
}

// pointer of a contiguous device tensor of `type`
void *dense(const at::Tensor &t, at::ScalarType type, const char *name)
{
    if (!t.is_cuda() || t.scalar_type() != type || !t.is_contiguous()) type_error(name, type_name(type));
    return t.data_ptr();
}
void *dense(PyObject *o, at::ScalarType type, const char *name)
{
    return o == Py_None ? nullptr : dense(tensor(o, name), type, name);
}

// pointer and row pitch of a 2-D uint8 device tensor with contiguous rows that may be spaced apart
struct Rows {
    uint8_t *p;
    int64_t pitch;
};
Rows rows(const at::Tensor &t, const char *name)
{
    if (!t.is_cuda() || t.scalar_type() != at::kByte || t.dim() != 2 || !(t.size(1) == 1 || t.stride(1) == 1) ||
        !(t.size(0) == 1 || t.stride(0) >= t.size(1)))
        type_error(name, "a 2-D device tensor of torch.uint8 with contiguous rows");
    return {static_cast<uint8_t *>(t.data_ptr()), t.size(0) > 1 ? t.stride(0) : t.size(1)};
}

// pointer of an operand that a kernel reads as many elements of as `x` has
void *dense_like(PyObject *o, at::ScalarType type, const char *name, const at::Tensor &x)
{
    if (o == Py_None) return nullptr;
    const at::Tensor &t = tensor(o, name);
    void *const p = dense(t, type, name);
    if (t.numel() < x.numel()) shape_error(name, t.sizes(), x.sizes());
    return p;
}

at::Tensor fresh(at::IntArrayRef shape, at::ScalarType type, const at::Tensor &like)
{
    return at::Tensor(at::detail::empty_cuda(shape, type, like.device(), std::nullopt));
}

// the caller's `out` (the kernels write shape-many elements: of that shape, or, without check_shape, any tensor that
// holds as many), or a new tensor
struct Out {
    at::Tensor t;
    PyObject *given = nullptr; // returned as it came
    PyObject *release()
    {
        if (given) {
            Py_INCREF(given);
            return given;
        }
        return THPVariable_Wrap(std::move(t));
    }
};
Out output(PyObject *o, at::IntArrayRef shape, at::ScalarType type, const at::Tensor &like, bool check_shape = true)
{
    Out out;
    if (o == Py_None) {
        out.t = fresh(shape, type, like);
    } else {
        out.t = tensor(o, "out");
        out.given = o;
        if (check_shape ? out.t.sizes() != shape : out.t.numel() < c10::multiply_integers(shape)) shape_error("out", out.t.sizes(), shape);
    }
    return out;
}

// scratch memory of a dense call: the caller's tensor, else a fresh one of the size the library asks for (it
// may go back to the allocator when the call has been enqueued: torch hands memory out in stream order)
struct Workspace {
    at::Tensor t;
    void *p = nullptr;
    size_t bytes = 0;
};
template <class Query> Workspace workspace(PyObject *o, const at::Tensor &like, bool required, Query query)
{
    Workspace w;
    if (o != Py_None) {
        const at::Tensor &t = tensor(o, "workspace");
        if (!t.is_cuda() || t.scalar_type() != at::kByte || !t.is_contiguous()) type_error("workspace", "a contiguous uint8 device tensor");
        w.p = t.data_ptr(), w.bytes = (size_t)t.numel();
        return w;
    }
    w.bytes = query();
    if (w.bytes) {
        try {
            w.t = fresh({(int64_t)w.bytes}, at::kByte, like);
            w.p = w.t.data_ptr();
        } catch (const c10::OutOfMemoryError &) {
            if (required) throw;
            w.bytes = 0; // padded copies can be as large as the operands: without room for them the library takes another route
        }
    }
    return w;
}

void *stream() { return c10::hip::getCurrentHIPStream().stream(); }

// the interpreter lock is given up for the lifetime of this object, however the scope is left
struct Unlocked {
    PyThreadState *const state = PyEval_SaveThread();
    Unlocked() = default;
    Unlocked(const Unlocked &) = delete;
    ~Unlocked() { PyEval_RestoreThread(state); }
};

// calls the library without the interpreter lock and raises for a status other than QNN_OK; the stream is looked up
// with the lock held, since that may throw
template <class F> void call(const char *name, F f)
{
    void *const s = stream();
    const qnn_status st = [&] {
        const Unlocked unlocked;
        return f(s);
    }();
    if (st == QNN_OK) return;
    PyObject *r = PyObject_CallFunction(g_check, "si", name, (int)st);
    if (r) {
        Py_DECREF(r);
        PyErr_Format(PyExc_RuntimeError, "%s failed with status %d", name, (int)st);
    }
    throw PythonErrorSet{};
}

using Args = PyObject *const *;

template <PyObject *(*F)(Args)> PyObject *guarded(PyObject *, Args a, Py_ssize_t)
{
    try {
        return F(a);
    } catch (const PythonErrorSet &) {
    } catch (...) {
        torch::translate_exception_to_python(std::current_exception());
    }
    return nullptr;
}
template <PyObject *(*F)(Args), int N> PyObject *entry(PyObject *self, Args a, Py_ssize_t n)
{
    if (n != N) {
        PyErr_Format(PyExc_TypeError, "expected %d arguments, got %zd", N, n);
        return nullptr;
    }
    return guarded<F>(self, a, n);
}

// ------------------------------------------------------------------------------- element-wise functions

template <bool WIDE> PyObject *f_quantize(Args a) // x, scale, zero_point, qmin, qmax, out
{
    const at::Tensor &x = tensor(a[0], "x");
    const auto *px = static_cast<const float *>(dense(x, at::kFloat, "x"));
    Out q = output(a[5], x.sizes(), WIDE ? at::kUInt16 : at::kByte, x);
    void *pq = dense(q.t, WIDE ? at::kUInt16 : at::kByte, "q");
    const size_t n = (size_t)x.numel();
    const float scale = real(a[1]);
    const int32_t z = i32(a[2]), lo = i32(a[3]), hi = i32(a[4]);
    if (WIDE) call("qnn_quantize_u16", [&](void *s) { return qnn_quantize_u16(px, static_cast<uint16_t *>(pq), n, scale, z, lo, hi, s); });
    else call("qnn_quantize", [&](void *s) { return qnn_quantize(px, static_cast<uint8_t *>(pq), n, scale, z, lo, hi, s); });
    return q.release();
}

template <bool WIDE> PyObject *f_dequantize(Args a) // q, scale, zero_point, out
{
    const at::Tensor &q = tensor(a[0], "q");
    const void *pq = dense(q, WIDE ? at::kUInt16 : at::kByte, "q");
    Out x = output(a[3], q.sizes(), at::kFloat, q, WIDE);
    auto *px = static_cast<float *>(dense(x.t, at::kFloat, "x"));
    const size_t n = (size_t)q.numel();
    const float scale = real(a[1]);
    const int32_t z = i32(a[2]);
    if (WIDE) call("qnn_dequantize_u16", [&](void *s) { return qnn_dequantize_u16(static_cast<const uint16_t *>(pq), px, n, scale, z, s); });
    else call("qnn_dequantize", [&](void *s) { return qnn_dequantize(static_cast<const uint8_t *>(pq), px, n, scale, z, s); });
    return x.release();
}

PyObject *f_requantize(Args a) // acc, mult, shift, per_channel, z_out, act_min, act_max, out
{
    const at::Tensor &acc = tensor(a[0], "acc");
    if (acc.dim() != 2) type_error("acc", "a 2-D tensor [rows, channels]");
    const auto *pa = static_cast<const int32_t *>(dense(acc, at::kInt, "acc"));
    Out y = output(a[7], acc.sizes(), at::kByte, acc);
    auto *py = static_cast<uint8_t *>(dense(y.t, at::kByte, "y"));
    const auto *mult = static_cast<const int32_t *>(dense(a[1], at::kInt, "mult"));
    const auto *shift = static_cast<const int32_t *>(dense(a[2], at::kInt, "shift"));
    const int per_channel = PyObject_IsTrue(a[3]);
    if (per_channel < 0) throw PythonErrorSet{};
    const int32_t z = i32(a[4]), lo = i32(a[5]), hi = i32(a[6]);
    call("qnn_requantize", [&](void *s) {
        return qnn_requantize(pa, py, (size_t)acc.size(0), (size_t)acc.size(1), mult, shift, per_channel, z, lo, hi, s);
    });
    return y.release();
}

// the entries of a qadd_params() dictionary
struct AddDict {
    int32_t v[P_COUNT];
};
AddDict add_dict(PyObject *o)
{
    AddDict d;
    for (int i = 0; i < P_COUNT; ++i) {
        if (PyDict_CheckExact(o)) {
            PyObject *item = PyDict_GetItemWithError(o, g_param_names[i]);
            if (!item) {
                if (!PyErr_Occurred()) PyErr_SetObject(PyExc_KeyError, g_param_names[i]);
                throw PythonErrorSet{};
            }
            d.v[i] = i32(item);
        } else {
            PyObject *item = PyObject_GetItem(o, g_param_names[i]);
            if (!item) throw PythonErrorSet{};
            const int64_t v = (int64_t)PyLong_AsUnsignedLongLongMask(item);
            Py_DECREF(item);
            if (v == -1 && PyErr_Occurred()) throw PythonErrorSet{};
            d.v[i] = (int32_t)v;
        }
    }
    return d;
}

PyObject *f_qadd(Args a) // a, z_a, b, z_b, params, z_out, act_min, act_max, out
{
    const at::Tensor &x = tensor(a[0], "a");
    const auto *pa = static_cast<const uint8_t *>(dense(x, at::kByte, "a"));
    Out y = output(a[8], x.sizes(), at::kByte, x);
    const AddDict d = add_dict(a[4]);
    const auto *pb = static_cast<const uint8_t *>(dense_like(a[2], at::kByte, "b", x));
    auto *py = static_cast<uint8_t *>(dense(y.t, at::kByte, "y"));
    const int32_t za = i32(a[1]), zb = i32(a[3]), z = i32(a[5]), lo = i32(a[6]), hi = i32(a[7]);
    call("qnn_qadd", [&](void *s) {
        return qnn_qadd(pa, za, d.v[P_MULT_A], d.v[P_SHIFT_A], pb, zb, d.v[P_MULT_B], d.v[P_SHIFT_B], d.v[P_LEFT], d.v[P_MULT_O],
                        d.v[P_SHIFT_O], z, lo, hi, py, (size_t)x.numel(), s);
    });
    return y.release();
}

PyObject *f_rescale_u8(Args a) // x, z_in, mult, shift, z_out, act_min, act_max, out
{
    const at::Tensor &x = tensor(a[0], "x");
    if (x.dim() != 2) type_error("x", "a 2-D device tensor of torch.uint8 with contiguous rows");
    const Rows rx = rows(x, "x");
    Out y = output(a[7], x.sizes(), at::kByte, x);
    const Rows ry = rows(y.t, "y");
    const int32_t zi = whole(a[1]), mult = whole(a[2]), shift = whole(a[3]), z = whole(a[4]), lo = whole(a[5]), hi = whole(a[6]);
    call("qnn_rescale_u8", [&](void *s) {
        return qnn_rescale_u8(rx.p, rx.pitch, zi, mult, shift, z, lo, hi, ry.p, ry.pitch, x.size(0), x.size(1), s);
    });
    return y.release();
}

qnn_dyn_qparams *range_state(PyObject *o) { return static_cast<qnn_dyn_qparams *>(dense(o, at::kInt, "state")); }

PyObject *f_minmax(Args a) // x, state, momentum, bits
{
    const at::Tensor &x = tensor(a[0], "x");
    const auto *px = static_cast<const float *>(dense(x, at::kFloat, "x"));
    qnn_dyn_qparams *st = range_state(a[1]);
    const float momentum = real(a[2]);
    const int bits = whole(a[3]);
    call("qnn_minmax", [&](void *s) { return qnn_minmax(px, (size_t)x.numel(), momentum, bits, st, s); });
    Py_INCREF(a[1]);
    return a[1];
}

template <bool DYNAMIC> PyObject *f_quantize_state(Args a) // x, state, out
{
    const at::Tensor &x = tensor(a[0], "x");
    const auto *px = static_cast<const float *>(dense(x, at::kFloat, "x"));
    Out q = output(a[2], x.sizes(), at::kByte, x);
    auto *pq = static_cast<uint8_t *>(dense(q.t, at::kByte, "q"));
    qnn_dyn_qparams *st = range_state(a[1]);
    if (DYNAMIC) call("qnn_quantize_dynamic", [&](void *s) { return qnn_quantize_dynamic(px, pq, (size_t)x.numel(), st, s); });
    else call("qnn_quantize_with", [&](void *s) { return qnn_quantize_with(px, pq, (size_t)x.numel(), st, s); });
    return q.release();
}

PyObject *f_simquant(Args a) // x, scale, zero_point, qmin, qmax, out
{
    const at::Tensor &x = tensor(a[0], "x");
    const auto *px = static_cast<const float *>(dense(x, at::kFloat, "x"));
    Out y = output(a[5], x.sizes(), at::kFloat, x, false);
    auto *py = static_cast<float *>(dense(y.t, at::kFloat, "y"));
    const float scale = real(a[1]);
    const int32_t z = whole(a[2]), lo = whole(a[3]), hi = whole(a[4]);
    call("qnn_simquant", [&](void *s) { return qnn_simquant(px, py, (size_t)x.numel(), scale, z, lo, hi, s); });
    return y.release();
}

PyObject *f_simquant_backward(Args a) // x, grad_y, scale, zero_point, qmin, qmax, out
{
    const at::Tensor &x = tensor(a[0], "x");
    const auto *px = static_cast<const float *>(dense(x, at::kFloat, "x"));
    Out g = output(a[6], x.sizes(), at::kFloat, x, false);
    const auto *pg = static_cast<const float *>(dense_like(a[1], at::kFloat, "grad_y", x));
    auto *po = static_cast<float *>(dense(g.t, at::kFloat, "grad_x"));
    const float scale = real(a[2]);
    const int32_t z = whole(a[3]), lo = whole(a[4]), hi = whole(a[5]);
    call("qnn_simquant_backward", [&](void *s) { return qnn_simquant_backward(px, pg, po, (size_t)x.numel(), scale, z, lo, hi, s); });
    return g.release();
}

// ------------------------------------------------------------------------------- matrix products

// the per-column parameters that every layer takes
struct Channels {
    const int32_t *bias, *mult, *shift;
};
Channels channels(PyObject *bias, PyObject *mult, PyObject *shift)
{
    return {static_cast<const int32_t *>(dense(bias, at::kInt, "bias")), static_cast<const int32_t *>(dense(mult, at::kInt, "mult")),
            static_cast<const int32_t *>(dense(shift, at::kInt, "shift"))};
}

// A and B of a product and its sizes
struct Product {
    const at::Tensor &A;
    Rows a;
    const void *b;
    int64_t M, N, K, ldb;
    int bits;
};
Product product(PyObject *oa, PyObject *ob, int bits, int layout)
{
    const at::Tensor &A = tensor(oa, "A"), &B = tensor(ob, "B");
    if (A.dim() != 2) type_error("A", "a 2-D device tensor of torch.uint8 with contiguous rows");
    if (B.dim() != 2) type_error("B", "a 2-D device tensor");
    const void *pb = dense(B, bits == 4 ? at::kByte : at::kChar, "B");
    int64_t N = B.size(0), ldb = B.size(1);
    if (bits == 4) ldb *= 2;
    else if (layout != QNN_B_COLUMNS_CONTIGUOUS) N = ldb = B.size(1);
    return {A, rows(A, "A"), pb, A.size(0), N, A.size(1), ldb, bits};
}
Workspace gemm_workspace(PyObject *o, const Product &p, bool asym)
{
    return workspace(o, p.A, asym, [&] { return qnn_qgemm_workspace_bytes(p.M, p.N, p.K, p.bits, asym); });
}

PyObject *f_qgemm(Args a) // A, z_a, B, mult, shift, z_out, act_min, act_max, bias, weight_bits, b_layout, out, workspace
{
    const int bits = i32(a[9]), layout = i32(a[10]);
    const Product p = product(a[0], a[2], bits, layout);
    Out c = output(a[11], {p.M, p.N}, at::kByte, p.A);
    const Rows rc = rows(c.t, "C");
    const Channels ch = channels(a[8], a[3], a[4]);
    const Workspace ws = gemm_workspace(a[12], p, false);
    const int32_t za = i32(a[1]), z = i32(a[5]), lo = i32(a[6]), hi = i32(a[7]);
    call("qnn_qgemm", [&](void *s) {
        return qnn_qgemm(p.a.p, p.a.pitch, za, p.b, p.ldb, layout, bits, p.M, p.N, p.K, ch.bias, ch.mult, ch.shift, z, lo, hi, rc.p, rc.pitch,
                         ws.p, ws.bytes, s);
    });
    return c.release();
}

PyObject *f_qgemm_noalloc(Args a) // A, z_a, B, mult, shift, z_out, act_min, act_max, out, bias, weight_bits
{
    const int bits = i32(a[10]);
    const Product p = product(a[0], a[2], bits, QNN_B_COLUMNS_CONTIGUOUS);
    const at::Tensor &out = tensor(a[8], "out");
    const int64_t want[2] = {p.M, p.N};
    if (out.sizes() != at::IntArrayRef(want, 2)) shape_error("out", out.sizes(), at::IntArrayRef(want, 2));
    const Rows rc = rows(out, "C");
    const Channels ch = channels(a[9], a[3], a[4]);
    const int32_t za = i32(a[1]), z = i32(a[5]), lo = i32(a[6]), hi = i32(a[7]);
    call("qnn_qgemm_noalloc", [&](void *s) {
        return qnn_qgemm_noalloc(p.a.p, p.a.pitch, za, p.b, p.ldb, QNN_B_COLUMNS_CONTIGUOUS, bits, p.M, p.N, p.K, ch.bias, ch.mult, ch.shift,
                                 z, lo, hi, rc.p, rc.pitch, s);
    });
    Py_INCREF(a[8]);
    return a[8];
}

qnn_add_params add_params(PyObject *dict, PyObject *z_r, PyObject *z_out, PyObject *act_min, PyObject *act_max)
{
    // operand a of the add is the layer's own result, operand b the residual
    const AddDict d = add_dict(dict);
    return {d.v[P_MULT_A], d.v[P_SHIFT_A], i32(z_r), d.v[P_MULT_B], d.v[P_SHIFT_B], d.v[P_LEFT], d.v[P_MULT_O], d.v[P_SHIFT_O],
            i32(z_out), i32(act_min), i32(act_max)};
}

// A, z_a, B, mult, shift, z_mid, mid_min, mid_max, residual, z_r, params, z_out, act_min, act_max, bias, weight_bits, out, workspace
PyObject *f_qgemm_add(Args a)
{
    const int bits = i32(a[15]);
    const Product p = product(a[0], a[2], bits, QNN_B_COLUMNS_CONTIGUOUS);
    Out c = output(a[16], {p.M, p.N}, at::kByte, p.A);
    const Rows rc = rows(c.t, "C"), rr = rows(tensor(a[8], "residual"), "residual");
    const qnn_add_params add = add_params(a[10], a[9], a[11], a[12], a[13]);
    const Channels ch = channels(a[14], a[3], a[4]);
    const Workspace ws = gemm_workspace(a[17], p, false);
    const int32_t za = i32(a[1]), z = i32(a[5]), lo = i32(a[6]), hi = i32(a[7]);
    call("qnn_qgemm_add", [&](void *s) {
        return qnn_qgemm_add(p.a.p, p.a.pitch, za, p.b, p.ldb, QNN_B_COLUMNS_CONTIGUOUS, bits, p.M, p.N, p.K, ch.bias, ch.mult, ch.shift, z, lo,
                             hi, rr.p, rr.pitch, &add, rc.p, rc.pitch, ws.p, ws.bytes, s);
    });
    return c.release();
}

PyObject *f_qgemm_asym(Args a) // A, z_a, B, z_w, mult, shift, z_out, act_min, act_max, bias, weight_bits, out, workspace
{
    const int bits = i32(a[10]);
    const Product p = product(a[0], a[2], bits, QNN_B_COLUMNS_CONTIGUOUS);
    Out c = output(a[11], {p.M, p.N}, at::kByte, p.A);
    const Rows rc = rows(c.t, "C");
    const auto *zw = static_cast<const int32_t *>(dense(a[3], at::kInt, "z_w"));
    const Channels ch = channels(a[9], a[4], a[5]);
    const Workspace ws = gemm_workspace(a[12], p, true);
    const int32_t za = i32(a[1]), z = i32(a[6]), lo = i32(a[7]), hi = i32(a[8]);
    call("qnn_qgemm_asym", [&](void *s) {
        return qnn_qgemm_asym(p.a.p, p.a.pitch, za, p.b, p.ldb, QNN_B_COLUMNS_CONTIGUOUS, bits, zw, p.M, p.N, p.K, ch.bias, ch.mult, ch.shift, z,
                              lo, hi, rc.p, rc.pitch, ws.p, ws.bytes, s);
    });
    return c.release();
}

PyObject *f_pack_b(Args a) // B_rows
{
    const at::Tensor &b = tensor(a[0], "B");
    if (b.dim() != 2) type_error("B", "a 2-D device tensor of torch.int8");
    const int64_t K = b.size(0), N = b.size(1);
    const auto *src = static_cast<const int8_t *>(dense(b, at::kChar, "B"));
    at::Tensor out = fresh({N, K}, at::kChar, b);
    auto *dst = static_cast<int8_t *>(out.data_ptr());
    call("qnn_pack_b", [&](void *s) { return qnn_pack_b(src, N, K, N, dst, K, s); });
    return THPVariable_Wrap(std::move(out));
}

// ------------------------------------------------------------------------------- convolutions

struct Conv {
    const at::Tensor &x;
    const uint8_t *px;
    const void *pw;
    int N, H, W, Cin, Cout, kh, kw, bits;
    Pair s, p;
    int64_t out[4];
    at::IntArrayRef shape() const { return at::IntArrayRef(out, 4); }
};
int64_t out_size(int64_t h, int k, int stride, int pad)
{
    if (stride <= 0) return 0; // the library rejects it
    const int64_t v = h + 2 * (int64_t)pad - k;
    return v < 0 ? 0 : v / stride + 1;
}
Conv conv(PyObject *ox, PyObject *ow, PyObject *stride, PyObject *pad, int bits, bool depthwise)
{
    const at::Tensor &x = tensor(ox, "x"), &w = tensor(ow, "w");
    if (x.dim() != 4) type_error("x", "a 4-D NHWC tensor");
    const int d = depthwise ? 0 : 1; // kh and kw are all that is looked at: a single channel may have [kh, kw]
    if (w.dim() < d + 2) type_error("w", depthwise ? "a weight tensor [kh, kw, C]" : "a weight tensor [Cout, kh, kw, Cin]");
    Conv c{x,
           static_cast<const uint8_t *>(dense(x, at::kByte, "x")),
           dense(w, bits == 4 ? at::kByte : at::kChar, "w"),
           (int)x.size(0),
           (int)x.size(1),
           (int)x.size(2),
           (int)x.size(3),
           (int)(depthwise ? x.size(3) : w.size(0)),
           (int)w.size(d),
           (int)w.size(d + 1),
           bits,
           pair(stride),
           pair(pad),
           {0, 0, 0, 0}};
    c.out[0] = c.N, c.out[1] = out_size(c.H, c.kh, c.s.h, c.p.h), c.out[2] = out_size(c.W, c.kw, c.s.w, c.p.w), c.out[3] = c.Cout;
    return c;
}
Workspace conv_workspace(PyObject *o, const Conv &c, bool asym)
{
    return workspace(o, c.x, asym, [&] {
        return qnn_qconv2d_workspace_bytes(c.N, c.H, c.W, c.Cin, c.Cout, c.kh, c.kw, c.bits, c.s.h, c.s.w, c.p.h, c.p.w, asym);
    });
}

PyObject *f_qconv2d(Args a) // x, z_x, w, stride, pad, mult, shift, z_out, act_min, act_max, bias, weight_bits, out, workspace
{
    const Conv c = conv(a[0], a[2], a[3], a[4], i32(a[11]), false);
    Out y = output(a[12], c.shape(), at::kByte, c.x);
    auto *py = static_cast<uint8_t *>(dense(y.t, at::kByte, "y"));
    const Channels ch = channels(a[10], a[5], a[6]);
    const Workspace ws = conv_workspace(a[13], c, false);
    const int32_t zx = i32(a[1]), z = i32(a[7]), lo = i32(a[8]), hi = i32(a[9]);
    call("qnn_qconv2d", [&](void *s) {
        return qnn_qconv2d(c.px, c.N, c.H, c.W, c.Cin, zx, c.pw, c.Cout, c.kh, c.kw, c.bits, c.s.h, c.s.w, c.p.h, c.p.w, ch.bias, ch.mult,
                           ch.shift, z, lo, hi, py, ws.p, ws.bytes, s);
    });
    return y.release();
}

// x, z_x, w, stride, pad, mult, shift, z_mid, mid_min, mid_max, residual, z_r, params, z_out, act_min, act_max, bias, weight_bits, out,
// workspace
PyObject *f_qconv2d_add(Args a)
{
    const Conv c = conv(a[0], a[2], a[3], a[4], i32(a[17]), false);
    Out y = output(a[18], c.shape(), at::kByte, c.x);
    const at::Tensor &res = tensor(a[10], "residual");
    if (res.sizes() != c.shape()) shape_error("residual", res.sizes(), c.shape());
    const auto *pr = static_cast<const uint8_t *>(dense(res, at::kByte, "residual"));
    auto *py = static_cast<uint8_t *>(dense(y.t, at::kByte, "y"));
    const qnn_add_params add = add_params(a[12], a[11], a[13], a[14], a[15]);
    const Channels ch = channels(a[16], a[5], a[6]);
    const Workspace ws = conv_workspace(a[19], c, false);
    const int32_t zx = i32(a[1]), z = i32(a[7]), lo = i32(a[8]), hi = i32(a[9]);
    call("qnn_qconv2d_add", [&](void *s) {
        return qnn_qconv2d_add(c.px, c.N, c.H, c.W, c.Cin, zx, c.pw, c.Cout, c.kh, c.kw, c.bits, c.s.h, c.s.w, c.p.h, c.p.w, ch.bias, ch.mult,
                               ch.shift, z, lo, hi, pr, &add, py, ws.p, ws.bytes, s);
    });
    return y.release();
}

PyObject *f_qconv2d_asym(Args a) // x, z_x, w, z_w, stride, pad, mult, shift, z_out, act_min, act_max, bias, weight_bits, out, workspace
{
    const Conv c = conv(a[0], a[2], a[4], a[5], i32(a[12]), false);
    Out y = output(a[13], c.shape(), at::kByte, c.x);
    auto *py = static_cast<uint8_t *>(dense(y.t, at::kByte, "y"));
    const auto *zw = static_cast<const int32_t *>(dense(a[3], at::kInt, "z_w"));
    const Channels ch = channels(a[11], a[6], a[7]);
    const Workspace ws = conv_workspace(a[14], c, true);
    const int32_t zx = i32(a[1]), z = i32(a[8]), lo = i32(a[9]), hi = i32(a[10]);
    call("qnn_qconv2d_asym", [&](void *s) {
        return qnn_qconv2d_asym(c.px, c.N, c.H, c.W, c.Cin, zx, c.pw, c.Cout, c.kh, c.kw, c.bits, zw, c.s.h, c.s.w, c.p.h, c.p.w, ch.bias,
                                ch.mult, ch.shift, z, lo, hi, py, ws.p, ws.bytes, s);
    });
    return y.release();
}

PyObject *f_qdwconv2d(Args a) // x, z_x, w, stride, pad, mult, shift, z_out, act_min, act_max, bias, out
{
    const Conv c = conv(a[0], a[2], a[3], a[4], 8, true);
    Out y = output(a[11], c.shape(), at::kByte, c.x);
    auto *py = static_cast<uint8_t *>(dense(y.t, at::kByte, "y"));
    const Channels ch = channels(a[10], a[5], a[6]);
    const int32_t zx = i32(a[1]), z = i32(a[7]), lo = i32(a[8]), hi = i32(a[9]);
    call("qnn_qdwconv2d", [&](void *s) {
        return qnn_qdwconv2d(c.px, c.N, c.H, c.W, c.Cin, zx, static_cast<const int8_t *>(c.pw), c.kh, c.kw, c.s.h, c.s.w, c.p.h, c.p.w, ch.bias,
                             ch.mult, ch.shift, z, lo, hi, py, s);
    });
    return y.release();
}

PyObject *f_qdwconv2d_asym(Args a) // x, z_x, w, z_w, stride, pad, mult, shift, z_out, act_min, act_max, bias, out
{
    const Conv c = conv(a[0], a[2], a[4], a[5], 8, true);
    Out y = output(a[12], c.shape(), at::kByte, c.x);
    auto *py = static_cast<uint8_t *>(dense(y.t, at::kByte, "y"));
    const auto *zw = static_cast<const int32_t *>(dense(a[3], at::kInt, "z_w"));
    const Channels ch = channels(a[11], a[6], a[7]);
    const int32_t zx = i32(a[1]), z = i32(a[8]), lo = i32(a[9]), hi = i32(a[10]);
    call("qnn_qdwconv2d_asym", [&](void *s) {
        return qnn_qdwconv2d_asym(c.px, c.N, c.H, c.W, c.Cin, zx, static_cast<const int8_t *>(c.pw), c.kh, c.kw, zw, c.s.h, c.s.w, c.p.h, c.p.w,
                                  ch.bias, ch.mult, ch.shift, z, lo, hi, py, s);
    });
    return y.release();
}

PyObject *f_set_check(Args a)
{
    Py_INCREF(a[0]);
    Py_XDECREF(g_check);
    g_check = a[0];
    Py_RETURN_NONE;
}

#define QNN_ENTRY(name, fn, n) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&entry<fn, n>)), METH_FASTCALL, nullptr}
PyMethodDef kMethods[] = {
    QNN_ENTRY("set_check", f_set_check, 1),
    QNN_ENTRY("quantize", f_quantize<false>, 6),
    QNN_ENTRY("quantize_u16", f_quantize<true>, 6),
    QNN_ENTRY("dequantize", f_dequantize<false>, 4),
    QNN_ENTRY("dequantize_u16", f_dequantize<true>, 4),
    QNN_ENTRY("requantize", f_requantize, 8),
    QNN_ENTRY("qadd", f_qadd, 9),
    QNN_ENTRY("rescale_u8", f_rescale_u8, 8),
    QNN_ENTRY("minmax", f_minmax, 4),
    QNN_ENTRY("quantize_with", f_quantize_state<false>, 3),
    QNN_ENTRY("quantize_dynamic", f_quantize_state<true>, 3),
    QNN_ENTRY("simquant", f_simquant, 6),
    QNN_ENTRY("simquant_backward", f_simquant_backward, 7),
    QNN_ENTRY("qgemm", f_qgemm, 13),
    QNN_ENTRY("qgemm_noalloc", f_qgemm_noalloc, 11),
    QNN_ENTRY("qgemm_add", f_qgemm_add, 18),
    QNN_ENTRY("qgemm_asym", f_qgemm_asym, 13),
    QNN_ENTRY("pack_b", f_pack_b, 1),
    QNN_ENTRY("qconv2d", f_qconv2d, 14),
    QNN_ENTRY("qconv2d_add", f_qconv2d_add, 20),
    QNN_ENTRY("qconv2d_asym", f_qconv2d_asym, 15),
    QNN_ENTRY("qdwconv2d", f_qdwconv2d, 12),
    QNN_ENTRY("qdwconv2d_asym", f_qdwconv2d_asym, 13),
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

} // namespace

PyMODINIT_FUNC PyInit__native(void)
{
    for (int i = 0; i < P_COUNT; ++i)
        if (!(g_param_names[i] = PyUnicode_InternFromString(kParamNames[i]))) return nullptr;
    return PyModule_Create(&kModule);
}
