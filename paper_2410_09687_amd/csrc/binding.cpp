// The calls of moin.py that a program makes per request or per layer, marshalled natively: what they check, allocate and
// pass on is what the Python text of these functions did before, in the same order.
//
// Bound by the host: a launch costs it 4 us, and beside its launches a call spent 4 to 6 us on ctypes' conversions, torch.empty
// and the interpreter's reads of shapes, types and addresses; here 1 to 2.  Us of host time, Python / native: moin_route 10.5 /
// 6.7 to 7.6, moin_lora_linear_planned of two launches 11.8 / 8.2 to 10, a decode layer's plan and four calls 71 / 40 to 49; where
// the kernels take less than that, a pass of the caller: one small step 27.6 / 21.7, one search and four merges 68 / 52.
#include <Python.h>

#include <ATen/ATen.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/tensor_dtypes.h>

#include "../../include/moin.h"

namespace {

PyObject *g_error = nullptr;   // moin.MoinError

constexpr int MAX_SHARED = 4;

// A Python exception has been set.
struct Raised {};

[[noreturn]] void fail(PyObject *type, const char *msg)
{
    PyErr_SetString(type, msg);
    throw Raised{};
}

const at::Tensor &tensor(PyObject *o, const char *name)
{
    if (!THPVariable_Check(o)) {
        PyErr_Format(PyExc_TypeError, "%s: tensor expected, got %s", name, Py_TYPE(o)->tp_name);
        throw Raised{};
    }
    return THPVariable_Unpack(o);
}

// Device address of a contiguous tensor on the GPU, of the given type.
void *dev_ptr(const at::Tensor &t, const char *name)
{
    if (!t.is_cuda()) {
        PyErr_Format(PyExc_ValueError, "%s must live on the GPU", name);
        throw Raised{};
    }
    if (!t.is_contiguous()) {
        PyErr_Format(PyExc_ValueError, "%s must be contiguous", name);
        throw Raised{};
    }
    return t.data_ptr();
}
void *dev_ptr(const at::Tensor &t, const char *name, at::ScalarType type)
{
    void *p = dev_ptr(t, name);
    if (t.scalar_type() != type) {
        PyErr_Format(PyExc_TypeError, "%s: expected %R, got %R", name, (PyObject *)torch::getTHPDtype(type),
                     (PyObject *)torch::getTHPDtype(t.scalar_type()));
        throw Raised{};
    }
    return p;
}
void *dev_ptr_or_null(PyObject *o, const char *name, at::ScalarType type)
{
    return o == Py_None ? nullptr : dev_ptr(tensor(o, name), name, type);
}

// Handles and streams: integers, None for null.
void *handle(PyObject *o)
{
    if (o == Py_None) return nullptr;
    void *p = PyLong_AsVoidPtr(o);
    if (!p && PyErr_Occurred()) throw Raised{};
    return p;
}
int64_t integer(PyObject *o)
{
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw Raised{};
    return v;
}
int32_t integer32(PyObject *o)
{
    const int64_t v = integer(o);
    if (v != (int32_t)v) fail(PyExc_OverflowError, "integer out of range");
    return (int32_t)v;
}
float real(PyObject *o)
{
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) throw Raised{};
    return (float)v;
}

int32_t size32(int64_t n)
{
    if (n != (int32_t)n) fail(PyExc_OverflowError, "dimension out of range");
    return (int32_t)n;
}

at::Tensor empty(at::IntArrayRef shape, at::ScalarType type, const at::Tensor &like)
{
    return at::empty(shape, at::TensorOptions().dtype(type).device(like.device()));
}

void check(int code, const char *what)
{
    if (code == 0) return;
    PyObject *e = g_error ? PyObject_CallFunction(g_error, "is", code, what) : nullptr;
    if (e) {
        PyErr_SetObject(g_error, e);
        Py_DECREF(e);
    } else if (!PyErr_Occurred()) {
        PyErr_SetString(PyExc_RuntimeError, what);
    }
    throw Raised{};
}
// The interpreter's lock, given back for the time of a call into the library and held again however that ends: what unwinds an
// exception drops references and sets Python's error.
struct Unlocked {
    PyThreadState *state = PyEval_SaveThread();
    Unlocked() = default;
    Unlocked(const Unlocked &) = delete;
    ~Unlocked() { PyEval_RestoreThread(state); }
};
template <class F>
void call(const char *what, F &&f)
{
    int code;
    {
        const Unlocked free;
        code = f();
    }
    check(code, what);
}

PyObject *wrapped(const at::Tensor &t)
{
    PyObject *o = THPVariable_Wrap(t);
    if (!o) throw Raised{};
    return o;
}
// Optional results: the caller's own object, a new tensor, or None.
struct Out {
    PyObject *own = nullptr;   // a reference of its own
    at::Tensor t;
    Out() = default;
    Out(Out &&o) noexcept : own(o.own), t(std::move(o.t)) { o.own = nullptr; }
    Out &operator=(Out &&o) noexcept
    {
        std::swap(own, o.own);
        t = std::move(o.t);
        return *this;
    }
    ~Out() { Py_XDECREF(own); }
    void is(PyObject *o)
    {
        Py_INCREF(o);
        own = o;
    }
    bool defined() const { return t.defined(); }
    PyObject *object() const
    {
        if (own) {
            Py_INCREF(own);
            return own;
        }
        if (t.defined()) return wrapped(t);
        Py_INCREF(Py_None);
        return Py_None;
    }
};
PyObject *tuple(const Out *o, int n)
{
    PyObject *r = PyTuple_New(n);
    if (!r) throw Raised{};
    for (int i = 0; i < n; ++i) {
        PyObject *v = nullptr;
        try {
            v = o[i].object();
        } catch (...) {
            Py_DECREF(r);
            throw;
        }
        PyTuple_SET_ITEM(r, i, v);
    }
    return r;
}

struct Search {
    const at::Tensor &emb, &cent;
    int64_t N;
    int32_t K, D;
    moin_dtype dt;
};
Search search(PyObject *e, PyObject *c)
{
    const at::Tensor &emb = tensor(e, "emb"), &cent = tensor(c, "centroids");
    if (emb.dim() != 2 || cent.dim() != 2 || emb.size(1) != cent.size(1))
        fail(PyExc_ValueError, "emb [N,D] and centroids [K,D] expected");
    if (emb.scalar_type() != cent.scalar_type() || (emb.scalar_type() != at::kFloat && emb.scalar_type() != at::kBFloat16))
        fail(PyExc_TypeError, "emb/centroids must both be float32 or both bfloat16");
    return Search{emb, cent, emb.size(0), size32(cent.size(0)), size32(emb.size(1)),
                  emb.scalar_type() == at::kBFloat16 ? MOIN_BF16 : MOIN_F32};
}
// (expert ids, centroid ids, counts): the caller's triple or new tensors
void triple(Out (&r)[3], const Search &s, PyObject *out, bool want_cids, bool want_counts, bool need_ids)
{
    if (out == Py_None) {
        r[0].t = empty({s.N}, at::kInt, s.cent);
        if (want_cids) r[1].t = empty({s.N}, at::kInt, s.cent);
        if (want_counts) r[2].t = empty({(int64_t)s.K}, at::kInt, s.cent);
        return;
    }
    PyObject *seq = PySequence_Fast(out, "out: a triple expected");
    if (!seq) throw Raised{};
    const bool three = PySequence_Fast_GET_SIZE(seq) == 3;
    if (three)
        for (int i = 0; i < 3; ++i) r[i].is(PySequence_Fast_GET_ITEM(seq, i));
    Py_DECREF(seq);
    if (!three) fail(PyExc_ValueError, "out: a triple expected");
    if (need_ids && r[0].own == Py_None) fail(PyExc_ValueError, "out: expert_ids is required");
    for (int i = 0; i < 3; ++i) {
        if (r[i].own == Py_None) continue;
        r[i].t = tensor(r[i].own, "out");
        if (r[i].t.scalar_type() != at::kInt || r[i].t.numel() != (i < 2 ? s.N : (int64_t)s.K))
            fail(PyExc_ValueError, "out: int32 tensors of N, N and K elements (or None) expected");
    }
}
int32_t *ids_ptr(const Out &o, const char *name, bool any = true)
{
    return o.defined() && any ? static_cast<int32_t *>(dev_ptr(o.t, name)) : nullptr;
}

// route(ctx, emb, centroids, slot, flags, want_centroid_ids, want_counts, stream, out, static)
PyObject *route(PyObject *const *a)
{
    const Search s = search(a[1], a[2]);
    Out r[3];
    triple(r, s, a[8], a[5] == Py_True, a[6] == Py_True, false);
    const bool fixed = a[9] == Py_True;
    moin_ctx *ctx = static_cast<moin_ctx *>(handle(a[0]));
    const void *emb = s.N ? dev_ptr(s.emb, "emb") : nullptr, *cent = dev_ptr(s.cent, "centroids");
    const int32_t *slot = static_cast<int32_t *>(dev_ptr_or_null(a[3], "slot_of_centroid", at::kInt));
    const uint32_t flags = (uint32_t)integer(a[4]);
    int32_t *eids = ids_ptr(r[0], "expert_ids", s.N > 0), *cids = ids_ptr(r[1], "centroid_ids", s.N > 0);
    int32_t *counts = ids_ptr(r[2], "counts");
    void *st = handle(a[7]);
    call(fixed ? "moin_route_static" : "moin_route", [&] {
        return (fixed ? moin_route_static : moin_route)(ctx, emb, cent, s.N, s.K, s.D, s.dt, slot, flags, eids, cids, counts, st);
    });
    return tuple(r, 3);
}

// route_topk(ctx, emb, centroids, k, slot, flags, stream)
PyObject *route_topk(PyObject *const *a)
{
    const Search s = search(a[1], a[2]);
    const int32_t k = integer32(a[3]);
    if (k < 1 || k > 8) fail(PyExc_ValueError, "k must be 1..8");
    Out r[3];
    r[0].t = empty({s.N, k}, at::kInt, s.cent);
    r[1].t = empty({s.N, k}, at::kInt, s.cent);
    r[2].t = empty({s.N, k}, at::kFloat, s.cent);
    moin_ctx *ctx = static_cast<moin_ctx *>(handle(a[0]));
    const void *emb = s.N ? dev_ptr(s.emb, "emb") : nullptr, *cent = dev_ptr(s.cent, "centroids");
    const int32_t *slot = static_cast<int32_t *>(dev_ptr_or_null(a[4], "slot_of_centroid", at::kInt));
    const uint32_t flags = (uint32_t)integer(a[5]);
    int32_t *eids = ids_ptr(r[0], "expert_ids", s.N > 0), *cids = ids_ptr(r[1], "centroid_ids", s.N > 0);
    float *d2 = s.N ? static_cast<float *>(dev_ptr(r[2].t, "dist2")) : nullptr;
    void *st = handle(a[6]);
    call("moin_route_topk", [&] { return moin_route_topk(ctx, emb, cent, s.N, s.K, s.D, s.dt, slot, flags, k, eids, cids, d2, st); });
    return tuple(r, 3);
}

const int32_t *rank_ptr(PyObject *o, int64_t E)
{
    if (o == Py_None) return nullptr;
    const at::Tensor &t = tensor(o, "rank_of_expert");
    if (t.numel() != E) fail(PyExc_ValueError, "rank_of_expert must have E entries");
    return static_cast<int32_t *>(dev_ptr(t, "rank_of_expert", at::kInt));
}
// (the count is checked first, the tensor itself where its turn comes)
void rank_count(PyObject *o, int64_t E)
{
    if (o != Py_None && tensor(o, "rank_of_expert").numel() != E)
        fail(PyExc_ValueError, "rank_of_expert must have E entries");
}

// route_plan(ctx, plan, emb, centroids, slot, flags, seq_offsets, T, E, ranks, want_centroid_ids, want_counts, stream, out)
PyObject *route_plan(PyObject *const *a)
{
    const Search s = search(a[2], a[3]);
    const at::Tensor &off = tensor(a[6], "seq_offsets");
    if (off.numel() != s.N + 1) fail(PyExc_ValueError, "seq_offsets must have N+1 entries");
    const int64_t T = integer(a[7]);
    const int32_t E = integer32(a[8]);
    rank_count(a[9], E);
    Out r[3];
    triple(r, s, a[13], a[10] == Py_True, a[11] == Py_True, true);
    moin_ctx *ctx = static_cast<moin_ctx *>(handle(a[0]));
    moin_plan *plan = static_cast<moin_plan *>(handle(a[1]));
    const void *emb = s.N ? dev_ptr(s.emb, "emb") : nullptr, *cent = dev_ptr(s.cent, "centroids");
    const int32_t *slot = static_cast<int32_t *>(dev_ptr_or_null(a[4], "slot_of_centroid", at::kInt));
    const uint32_t flags = (uint32_t)integer(a[5]);
    const int32_t *offs = static_cast<int32_t *>(dev_ptr(off, "seq_offsets", at::kInt)), *ranks = rank_ptr(a[9], E);
    int32_t *eids = ids_ptr(r[0], "expert_ids"), *cids = ids_ptr(r[1], "centroid_ids", s.N > 0), *counts = ids_ptr(r[2], "counts");
    void *st = handle(a[12]);
    call("moin_route_plan", [&] {
        return moin_route_plan(ctx, plan, emb, cent, s.N, s.K, s.D, s.dt, slot, flags, offs, T, E, ranks, eids, cids, counts, st);
    });
    return tuple(r, 3);
}

// plan_build(ctx, plan, seq_offsets, expert_ids, T, E, ranks, stream) -> S
PyObject *plan_build(PyObject *const *a)
{
    const at::Tensor &off = tensor(a[2], "seq_offsets"), &ids = tensor(a[3], "expert_ids");
    const int64_t S = ids.numel(), T = integer(a[4]);
    const int32_t E = integer32(a[5]);
    if (off.numel() != S + 1) fail(PyExc_ValueError, "seq_offsets must have S+1 entries");
    rank_count(a[6], E);
    moin_ctx *ctx = static_cast<moin_ctx *>(handle(a[0]));
    moin_plan *plan = static_cast<moin_plan *>(handle(a[1]));
    const int32_t *offs = static_cast<int32_t *>(dev_ptr(off, "seq_offsets", at::kInt));
    const int32_t *eids = S ? static_cast<int32_t *>(dev_ptr(ids, "expert_ids", at::kInt)) : nullptr, *ranks = rank_ptr(a[6], E);
    void *st = handle(a[7]);
    const int32_t S32 = size32(S);
    call("moin_plan_build_ranked", [&] { return moin_plan_build_ranked(ctx, plan, offs, eids, S32, T, E, ranks, st); });
    return PyLong_FromLongLong(S);
}

struct Dims {
    int32_t d_in, d_out, E, r;
};
Dims stack_dims(const at::Tensor &W, PyObject *A, PyObject *B)
{
    if (W.dim() != 2) fail(PyExc_ValueError, "W [d_out,d_in] expected");
    const int64_t d_out = W.size(0), d_in = W.size(1);
    if (A == Py_None || B == Py_None) return Dims{size32(d_in), size32(d_out), 0, 0};
    const at::Tensor &a = tensor(A, "A_stack"), &b = tensor(B, "B_stack");
    if (a.dim() != 3 || b.dim() != 3 || a.size(2) != d_in || b.size(0) != a.size(0) || b.size(1) != d_out || b.size(2) != a.size(1))
        fail(PyExc_ValueError, "A_stack [E,r,d_in] / B_stack [E,d_out,r] shape mismatch");
    return Dims{size32(d_in), size32(d_out), size32(a.size(0)), size32(a.size(1))};
}
at::ScalarType y_type(PyObject *o)
{
    const at::ScalarType t = THPDtype_Check(o) ? reinterpret_cast<THPDtype *>(o)->scalar_type : at::ScalarType::Undefined;
    if (t != at::kFloat && t != at::kBFloat16) fail(PyExc_TypeError, "y dtype must be bfloat16 or float32");
    return t;
}
Out y_out(const at::Tensor &x, int64_t d_out, at::ScalarType t, PyObject *out)
{
    Out y;
    if (out == Py_None) {
        y.t = empty({x.size(0), d_out}, t, x);
        return y;
    }
    y.is(out);
    y.t = tensor(out, "out");
    if (y.t.dim() != 2 || y.t.size(0) != x.size(0) || y.t.size(1) != d_out || y.t.scalar_type() != t)
        fail(PyExc_ValueError, "out has the wrong shape or dtype");
    return y;
}
moin_dtype y_enum(at::ScalarType t) { return t == at::kBFloat16 ? MOIN_BF16 : MOIN_F32; }

// lora_linear(ctx, x, seq_offsets, expert_ids, W, A, B, scale, y_dtype, out, stream, ranks)
PyObject *lora_linear(PyObject *const *a)
{
    const at::Tensor &x = tensor(a[1], "x"), &off = tensor(a[2], "seq_offsets"), &ids = tensor(a[3], "expert_ids"), &W = tensor(a[4], "W");
    if (x.dim() != 2 || W.dim() != 2 || x.size(1) != W.size(1)) fail(PyExc_ValueError, "x [T,d_in] and W [d_out,d_in] expected");
    const Dims d = stack_dims(W, a[5], a[6]);
    rank_count(a[11], d.E);
    const int64_t S = ids.numel(), T = x.size(0);
    if (off.numel() != S + 1) fail(PyExc_ValueError, "seq_offsets must have S+1 entries");
    const at::ScalarType yt = y_type(a[8]);
    Out y = y_out(x, d.d_out, yt, a[9]);
    moin_ctx *ctx = static_cast<moin_ctx *>(handle(a[0]));
    const void *px = T ? dev_ptr(x, "x", at::kBFloat16) : nullptr;
    const int32_t *offs = static_cast<int32_t *>(dev_ptr(off, "seq_offsets", at::kInt));
    const int32_t *eids = S ? static_cast<int32_t *>(dev_ptr(ids, "expert_ids", at::kInt)) : nullptr;
    const void *pW = dev_ptr(W, "W", at::kBFloat16), *pA = dev_ptr_or_null(a[5], "A_stack", at::kBFloat16);
    const void *pB = dev_ptr_or_null(a[6], "B_stack", at::kBFloat16);
    const int32_t *ranks = rank_ptr(a[11], d.E);
    const float scale = real(a[7]);
    void *py = T ? dev_ptr(y.t, "y") : nullptr, *st = handle(a[10]);
    const int32_t S32 = size32(S);
    if (ranks)
        call("moin_lora_linear_ranked", [&] {
            return moin_lora_linear_ranked(ctx, px, offs, eids, S32, T, pW, pA, pB, d.E, d.d_in, d.d_out, d.r, ranks, scale, py,
                                           y_enum(yt), st);
        });
    else
        call("moin_lora_linear", [&] {
            return moin_lora_linear(ctx, px, offs, eids, S32, T, pW, pA, pB, d.E, d.d_in, d.d_out, d.r, scale, py, y_enum(yt), st);
        });
    return y.object();
}

void planned_experts(const Dims &d, int64_t plan_E, const char *msg)
{
    if (d.E && d.E != plan_E) fail(PyExc_ValueError, msg);
}

// lora_linear_planned(ctx, plan, plan.T, plan.E, x, W, A, B, scale, y_dtype, out, stream)
PyObject *lora_linear_planned(PyObject *const *a)
{
    const at::Tensor &x = tensor(a[4], "x"), &W = tensor(a[5], "W");
    if (x.dim() != 2 || W.dim() != 2 || x.size(1) != W.size(1) || x.size(0) != integer(a[2]))
        fail(PyExc_ValueError, "x [T,d_in] (T as planned) and W [d_out,d_in] expected");
    const Dims d = stack_dims(W, a[6], a[7]);
    planned_experts(d, integer(a[3]), "stack holds a different number of experts than the plan was built for");
    const at::ScalarType yt = y_type(a[9]);
    const int64_t T = x.size(0);
    Out y = y_out(x, d.d_out, yt, a[10]);
    moin_ctx *ctx = static_cast<moin_ctx *>(handle(a[0]));
    const moin_plan *plan = static_cast<moin_plan *>(handle(a[1]));
    const void *px = T ? dev_ptr(x, "x", at::kBFloat16) : nullptr, *pW = dev_ptr(W, "W", at::kBFloat16);
    const void *pA = dev_ptr_or_null(a[6], "A_stack", at::kBFloat16), *pB = dev_ptr_or_null(a[7], "B_stack", at::kBFloat16);
    const float scale = real(a[8]);
    void *py = T ? dev_ptr(y.t, "y") : nullptr, *st = handle(a[11]);
    call("moin_lora_linear_planned", [&] {
        return moin_lora_linear_planned(ctx, plan, px, pW, pA, pB, d.d_in, d.d_out, d.r, scale, py, y_enum(yt), st);
    });
    return y.object();
}

// lora_linear_mx_planned(ctx, plan, plan.T, plan.E, x, Wq, Ws, A, B, scale, xq, xs, emit, y_dtype, out, stream)
PyObject *lora_linear_mx_planned(PyObject *const *a)
{
    const at::Tensor &x = tensor(a[4], "x"), &Wq = tensor(a[5], "Wq"), &Ws = tensor(a[6], "Ws");
    if (x.dim() != 2 || Wq.dim() != 2 || x.size(1) != Wq.size(1) || x.size(0) != integer(a[2]))
        fail(PyExc_ValueError, "x [T,d_in] (T as planned) and Wq [d_out,d_in] expected");
    if (Wq.scalar_type() != at::kByte || Ws.scalar_type() != at::kByte || Wq.size(1) % 128 || Ws.dim() != 3 ||
        Ws.size(0) != Wq.size(1) / 128 || Ws.size(1) != Wq.size(0) || Ws.size(2) != 4)
        fail(PyExc_ValueError, "Wq [d_out,d_in] / Ws [d_in/128,d_out,4] (blocked layout) uint8 expected");
    const Dims d = stack_dims(Wq, a[7], a[8]);
    planned_experts(d, integer(a[3]), "stack holds a different number of experts than the plan was built for");
    const int64_t T = x.size(0);
    const bool given = a[10] != Py_None, emit = a[12] == Py_True;
    if (given != (a[11] != Py_None)) fail(PyExc_ValueError, "xq and xs go together");
    if (given) {
        const at::Tensor &q = tensor(a[10], "xq"), &s = tensor(a[11], "xs");
        if (q.dim() != 2 || q.size(0) != T || q.size(1) != d.d_in || s.dim() != 3 || s.size(0) != d.d_in / 128 || s.size(1) != T ||
            s.size(2) != 4)
            fail(PyExc_ValueError, "xq [T,d_in] / xs [d_in/128,T,4] (blocked layout) expected");
    }
    if (emit && !given) fail(PyExc_ValueError, "emit=True needs xq and xs to write to");
    const int32_t mode = !given ? MOIN_MX_X_INTERNAL : emit ? MOIN_MX_X_EMIT : MOIN_MX_X_GIVEN;
    const at::ScalarType yt = y_type(a[13]);
    Out y = y_out(x, d.d_out, yt, a[14]);
    moin_ctx *ctx = static_cast<moin_ctx *>(handle(a[0]));
    const moin_plan *plan = static_cast<moin_plan *>(handle(a[1]));
    const void *px = T ? dev_ptr(x, "x", at::kBFloat16) : nullptr;
    void *pq = dev_ptr_or_null(a[10], "xq", at::kByte), *ps = dev_ptr_or_null(a[11], "xs", at::kByte);
    const void *pWq = dev_ptr(Wq, "Wq", at::kByte), *pWs = dev_ptr(Ws, "Ws", at::kByte);
    const void *pA = dev_ptr_or_null(a[7], "A_stack", at::kBFloat16), *pB = dev_ptr_or_null(a[8], "B_stack", at::kBFloat16);
    const float scale = real(a[9]);
    void *py = T ? dev_ptr(y.t, "y") : nullptr, *st = handle(a[15]);
    call("moin_lora_linear_mx_planned", [&] {
        return moin_lora_linear_mx_planned(ctx, plan, px, pq, ps, mode, pWq, pWs, pA, pB, d.d_in, d.d_out, d.r, scale, py,
                                           y_enum(yt), st);
    });
    return y.object();
}

// A sequence of n objects, held while the call runs.
struct Items {
    PyObject *seq = nullptr;
    int n = 0;
    explicit Items(PyObject *o, const char *msg)
    {
        if (o == Py_None) return;
        seq = PySequence_Fast(o, msg);
        if (!seq) throw Raised{};
        n = (int)PySequence_Fast_GET_SIZE(seq);
    }
    ~Items() { Py_XDECREF(seq); }
    Items(const Items &) = delete;
    PyObject *operator[](int i) const { return seq ? PySequence_Fast_GET_ITEM(seq, i) : Py_None; }
};

// lora_linear_planned_shared(ctx, plan, plan.T, plan.E, x, Ws, A_stacks, B_stacks, scale, y_dtype, outs, stream) -> list
PyObject *lora_linear_planned_shared(PyObject *const *a)
{
    const Items Ws(a[5], "Ws: a list expected"), As(a[6], "A_stacks: a list expected"), Bs(a[7], "B_stacks: a list expected"),
        outs(a[10], "outs: a list expected");
    const int n = Ws.n;
    if (n < 1 || n > MAX_SHARED) fail(PyExc_ValueError, "1 to 4 projections expected");
    if (!As.seq != !Bs.seq) fail(PyExc_ValueError, "A_stacks and B_stacks go together");
    if (As.seq && (As.n != n || Bs.n != n)) fail(PyExc_ValueError, "one A_stack and one B_stack per weight expected");
    if (outs.seq && outs.n < n) fail(PyExc_IndexError, "outs: one per weight expected");
    Dims d[MAX_SHARED];
    for (int i = 0; i < n; ++i) d[i] = stack_dims(tensor(Ws[i], "W"), As[i], Bs[i]);
    for (int i = 1; i < n; ++i)
        if (d[i].d_in != d[0].d_in || d[i].E != d[0].E || d[i].r != d[0].r)
            fail(PyExc_ValueError, "the projections must agree in d_in, E and r");
    const at::Tensor &x = tensor(a[4], "x");
    if (x.dim() != 2 || x.size(1) != d[0].d_in || x.size(0) != integer(a[2])) fail(PyExc_ValueError, "x [T,d_in] (T as planned) expected");
    planned_experts(d[0], integer(a[3]), "stacks hold a different number of experts than the plan was built for");
    const int64_t T = x.size(0);
    const at::ScalarType yt = y_type(a[9]);
    Out y[MAX_SHARED];
    for (int i = 0; i < n; ++i) y[i] = y_out(x, d[i].d_out, yt, outs[i]);
    moin_ctx *ctx = static_cast<moin_ctx *>(handle(a[0]));
    const moin_plan *plan = static_cast<moin_plan *>(handle(a[1]));
    const void *px = T ? dev_ptr(x, "x", at::kBFloat16) : nullptr;
    const void *pW[MAX_SHARED], *pA[MAX_SHARED], *pB[MAX_SHARED];
    void *py[MAX_SHARED];
    int32_t d_out[MAX_SHARED];
    for (int i = 0; i < n; ++i) pW[i] = dev_ptr(tensor(Ws[i], "W"), "W", at::kBFloat16);
    for (int i = 0; i < n; ++i) pA[i] = dev_ptr_or_null(As[i], "A_stack", at::kBFloat16);
    for (int i = 0; i < n; ++i) pB[i] = dev_ptr_or_null(Bs[i], "B_stack", at::kBFloat16);
    for (int i = 0; i < n; ++i) {
        d_out[i] = d[i].d_out;
        py[i] = T ? dev_ptr(y[i].t, "y") : nullptr;
    }
    const float scale = real(a[8]);
    void *st = handle(a[11]);
    call("moin_lora_linear_planned_shared", [&] {
        return moin_lora_linear_planned_shared(ctx, plan, px, n, pW, As.seq ? pA : nullptr, Bs.seq ? pB : nullptr, d[0].d_in, d_out,
                                               d[0].r, scale, py, y_enum(yt), st);
    });
    PyObject *list = PyList_New(n);
    if (!list) throw Raised{};
    for (int i = 0; i < n; ++i) {
        PyObject *v = nullptr;
        try {
            v = y[i].object();
        } catch (...) {
            Py_DECREF(list);
            throw;
        }
        PyList_SET_ITEM(list, i, v);
    }
    return list;
}

// merge_adapters(ctx, A, B, ids, weights, A_out, B_out, stream)
PyObject *merge_adapters(PyObject *const *a)
{
    const at::Tensor &A = tensor(a[1], "A_stack"), &B = tensor(a[2], "B_stack"), &ids = tensor(a[3], "ids"), &w = tensor(a[4], "weights");
    const at::Tensor &Ao = tensor(a[5], "A_out"), &Bo = tensor(a[6], "B_out");
    if (A.dim() != 3 || B.dim() != 3 || B.size(0) != A.size(0) || B.size(2) != A.size(1))
        fail(PyExc_ValueError, "A_stack [E,r,d_in] / B_stack [E,d_out,r] shape mismatch");
    const int64_t d_in = A.size(2), d_out = B.size(1), n = ids.numel();
    if (w.numel() != n) fail(PyExc_ValueError, "one weight per id expected");
    if (Ao.dim() != 2 || Bo.dim() != 2 || Ao.size(1) != d_in || Bo.size(0) != d_out || Bo.size(1) != Ao.size(0))
        fail(PyExc_ValueError, "A_out [r_out,d_in] / B_out [d_out,r_out] expected");
    moin_ctx *ctx = static_cast<moin_ctx *>(handle(a[0]));
    const void *pA = dev_ptr(A, "A_stack", at::kBFloat16), *pB = dev_ptr(B, "B_stack", at::kBFloat16);
    const int32_t *pi = static_cast<int32_t *>(dev_ptr(ids, "ids", at::kInt));
    const float *pw = static_cast<float *>(dev_ptr(w, "weights", at::kFloat));
    void *po = dev_ptr(Ao, "A_out", at::kBFloat16), *pb = dev_ptr(Bo, "B_out", at::kBFloat16), *st = handle(a[7]);
    const int32_t E = size32(A.size(0)), r = size32(A.size(1)), di = size32(d_in), dout = size32(d_out), n32 = size32(n),
                  r_out = size32(Ao.size(0));
    call("moin_merge_adapters", [&] { return moin_merge_adapters(ctx, pA, pB, E, r, di, dout, pi, pw, n32, r_out, po, pb, st); });
    Py_RETURN_NONE;
}

// set_error(type): what a status other than success is raised as
PyObject *set_error(PyObject *const *a)
{
    Py_INCREF(a[0]);
    Py_XDECREF(g_error);
    g_error = a[0];
    Py_RETURN_NONE;
}

// No C++ exception leaves through the interpreter.
template <PyObject *(*F)(PyObject *const *), int N>
PyObject *entry(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != N) {
        PyErr_Format(PyExc_TypeError, "%d arguments expected, got %zd", N, n);
        return nullptr;
    }
    try {
        return F(args);
    } catch (const Raised &) {
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}
#define MOIN_ENTRY(f, n) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(entry<f, n>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    MOIN_ENTRY(route, 10), MOIN_ENTRY(route_topk, 7), MOIN_ENTRY(route_plan, 14), MOIN_ENTRY(plan_build, 8),
    MOIN_ENTRY(lora_linear, 12), MOIN_ENTRY(lora_linear_planned, 12), MOIN_ENTRY(lora_linear_mx_planned, 16),
    MOIN_ENTRY(lora_linear_planned_shared, 12), MOIN_ENTRY(merge_adapters, 8), MOIN_ENTRY(set_error, 1),
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_moin_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__moin_binding() { return PyModule_Create(&module); }
