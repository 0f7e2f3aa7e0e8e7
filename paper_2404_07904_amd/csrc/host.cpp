// Native call path of the Python binding: unpacks the tensors of a call, allocates the outputs and the
// workspace the caller did not hand over, and calls the C ABI of libhgrn2.so on the current stream.
// It holds no state and no memory of its own (allocations go to the framework's caching allocator, as
// torch.empty's do) and does nothing the C ABI does not: every result comes from the HIP kernels.
//
// Why native: a decode step of one request runs 3.5 us on the GPU, and the same call made through
// ctypes (argument conversion, torch.empty, the stream lookup) keeps the host busy for 10 us; the
// small forward passes are bound the same way once their kernels take less than twenty.
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/hip/EmptyTensor.h>
#include <c10/hip/HIPStream.h>
#include <Python.h>

#include <algorithm>
#include <utility>

#include "../../include/hgrn2.h"

namespace {

PyObject* hgrn2_error = nullptr;          // binding.Hgrn2Error, set by set_error()

struct PyFail {};                         // a Python exception is set

[[noreturn]] void fail(PyObject* type, const char* msg)
{
    PyErr_SetString(type, msg);
    throw PyFail{};
}

void require(bool ok, const char* msg)
{
    if (!ok) fail(PyExc_AssertionError, msg);
}

// One positional argument: a tensor, or None where the entry point allows it.
const at::Tensor* maybe_tensor(PyObject* o)
{
    if (o == Py_None) return nullptr;
    if (!THPVariable_Check(o)) fail(PyExc_TypeError, "expected a tensor");
    return &THPVariable_Unpack(o);
}

const at::Tensor& tensor(PyObject* o)
{
    const at::Tensor* t = maybe_tensor(o);
    if (!t) fail(PyExc_TypeError, "expected a tensor, got None");
    return *t;
}

int32_t to_int(PyObject* o)
{
    const long x = PyLong_AsLong(o);
    if (x == -1 && PyErr_Occurred()) throw PyFail{};
    return (int32_t)x;
}

bool to_bool(PyObject* o)
{
    const int x = PyObject_IsTrue(o);
    if (x < 0) throw PyFail{};
    return x != 0;
}

int32_t dtype_of(const at::Tensor& t)
{
    if (t.scalar_type() == at::kBFloat16) return HGRN2_BF16;
    if (t.scalar_type() == at::kFloat) return HGRN2_F32;
    fail(PyExc_TypeError, "unsupported dtype");
}

void* ptr(const at::TensorBase& t)
{
    require(t.is_cuda() && t.is_contiguous(), "tensors must be contiguous device tensors");
    return t.data_ptr();
}
void* ptr(const at::Tensor* t) { return t ? ptr(*t) : nullptr; }
const float* fptr(const at::Tensor* t) { return static_cast<const float*>(ptr(t)); }

void* stream() { return c10::hip::getCurrentHIPStream().stream(); }

at::TensorBase fresh(at::IntArrayRef sizes, at::ScalarType dtype, const at::Tensor& like)
{
    require(like.is_cuda(), "tensors must be contiguous device tensors");
    return at::detail::empty_cuda(sizes, dtype, like.device(), std::nullopt);
}
at::TensorBase fresh_like(const at::Tensor& t) { return fresh(t.sizes(), t.scalar_type(), t); }

// the caller's buffer, or a fresh one
at::TensorBase given_or_like(const at::Tensor* given, const at::Tensor& like) { return given ? at::TensorBase(*given) : fresh_like(like); }

at::TensorBase workspace(const at::Tensor* given, size_t bytes, const at::Tensor& like)
{
    return given ? at::TensorBase(*given) : fresh({(int64_t)std::max<size_t>(bytes, 256)}, at::kByte, like);
}

void check_status(int rc, const char* name)
{
    if (rc == HGRN2_OK) return;
    PyObject* e = hgrn2_error ? PyObject_CallFunction(hgrn2_error, "is", rc, name) : nullptr;
    if (e) {
        PyErr_SetObject(hgrn2_error, e);
        Py_DECREF(e);
    } else if (!PyErr_Occurred()) {
        PyErr_Format(PyExc_RuntimeError, "%s failed with status %d", name, rc);
    }
    throw PyFail{};
}

// Runs an entry point without the interpreter lock.
template <typename F> void enqueue(const char* name, F call)
{
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = call();
    Py_END_ALLOW_THREADS
    check_status(rc, name);
}

// The results as a tuple (an undefined tensor is None).
template <typename... Ts> PyObject* tuple_of(Ts&&... ts)
{
    PyObject* r = PyTuple_New(sizeof...(ts));
    if (!r) throw PyFail{};
    Py_ssize_t i = 0;
    auto put = [&](at::TensorBase t) {
        PyObject* o;
        if (t.defined()) o = THPVariable_Wrap(std::move(t));
        else { Py_INCREF(Py_None); o = Py_None; }
        PyTuple_SET_ITEM(r, i++, o);
    };
    (put(std::forward<Ts>(ts)), ...);
    return r;
}

PyObject* wrap(at::TensorBase t) { return THPVariable_Wrap(std::move(t)); }

hgrn2_shape equal_shape(const at::Tensor& q, const at::Tensor& v, const at::Tensor& f, int32_t chunk, int32_t layout,
                        const at::Tensor* flag)
{
    if (q.dim() != 4 || v.dim() < 1) fail(PyExc_ValueError, "q, f, v must be 4-dimensional");
    hgrn2_shape s{};
    const bool bnhd = layout == HGRN2_LAYOUT_BNHD;
    s.B = (int32_t)q.size(0); s.H = (int32_t)q.size(bnhd ? 2 : 1); s.N = (int32_t)q.size(bnhd ? 1 : 2);
    s.dk = (int32_t)q.size(3); s.dv = (int32_t)v.size(-1);
    s.chunk = chunk; s.io_dtype = dtype_of(q); s.gate_dtype = dtype_of(f); s.layout = layout;
    if (flag) {
        require(flag->scalar_type() == at::kInt && flag->is_cuda() && flag->numel() >= 1, "domain_flag: a device int32");
        s.gate_domain_flag = static_cast<int32_t*>(flag->data_ptr());
    }
    return s;
}

hgrn2_shape packed_shape(const at::Tensor& q, const at::Tensor& v, const at::Tensor& f, const at::Tensor& cu, int32_t chunk,
                         const at::Tensor* flag)
{
    require(cu.scalar_type() == at::kInt && cu.is_contiguous(), "cu_seqlens: a contiguous int32 tensor");
    if (q.dim() != 3) fail(PyExc_ValueError, "q, f, v must be 3-dimensional");
    hgrn2_shape s{};
    s.B = (int32_t)cu.numel() - 1; s.H = (int32_t)q.size(1); s.N = (int32_t)q.size(0);
    s.dk = (int32_t)q.size(2); s.dv = (int32_t)v.size(-1);
    s.chunk = chunk; s.io_dtype = dtype_of(q); s.gate_dtype = dtype_of(f); s.layout = HGRN2_LAYOUT_BNHD;
    if (flag) {
        require(flag->scalar_type() == at::kInt && flag->is_cuda() && flag->numel() >= 1, "domain_flag: a device int32");
        s.gate_domain_flag = static_cast<int32_t*>(flag->data_ptr());
    }
    return s;
}

at::TensorBase state_tensor(const hgrn2_shape& s, const at::Tensor& like)
{
    return fresh({s.B, s.H, s.dk, s.dv}, at::kFloat, like);
}
at::TensorBase state_or_none(const at::Tensor* given, bool want, const hgrn2_shape& s, const at::Tensor& like)
{
    if (given) return *given;
    return want ? state_tensor(s, like) : at::TensorBase();
}
void* out_ptr(const at::TensorBase& t) { return t.defined() ? ptr(t) : nullptr; }
float* out_fptr(const at::TensorBase& t) { return static_cast<float*>(out_ptr(t)); }

void check_count(Py_ssize_t n, Py_ssize_t want)
{
    if (n != want) fail(PyExc_TypeError, "wrong number of arguments");
}

typedef PyObject* const* Args;

// step(q_t, f_t, None, v_t, state, o_t or None); step_gated(q_t, z_t, beta, v_t, state, o_t or None)
template <bool GATED> PyObject* step(Args a, Py_ssize_t n)
{
    check_count(n, 6);
    const at::Tensor& q = tensor(a[0]); const at::Tensor& f = tensor(a[1]); const at::Tensor* beta = maybe_tensor(a[2]);
    const at::Tensor& v = tensor(a[3]); const at::Tensor& state = tensor(a[4]); const at::Tensor* given = maybe_tensor(a[5]);
    if (q.dim() != 3) fail(PyExc_ValueError, "q_t must be 3-dimensional");
    const int32_t B = (int32_t)q.size(0), H = (int32_t)q.size(1), dk = (int32_t)q.size(2), dv = (int32_t)v.size(-1);
    require(state.scalar_type() == at::kFloat && state.dim() == 4 && state.size(0) == B && state.size(1) == H &&
            state.size(2) == dk && state.size(3) == dv, "state: fp32 [B, H, dk, dv]");
    if (GATED) require(beta && beta->scalar_type() == at::kFloat && beta->dim() == 2 && beta->size(0) == H && beta->size(1) == dk, "beta: fp32 [H, dk]");
    at::TensorBase o = given_or_like(given, v);
    const int32_t io = dtype_of(q), ge = dtype_of(f);
    const void *qp = ptr(q), *fp = ptr(f), *vp = ptr(v);
    const float* bp = fptr(beta);
    float* sp = static_cast<float*>(ptr(state));
    void *op = ptr(o), *st = stream();
    if (GATED) enqueue("hgrn2_step_gated", [&] { return hgrn2_step_gated(B, H, dk, dv, io, ge, qp, fp, bp, vp, sp, op, st); });
    else enqueue("hgrn2_step", [&] { return hgrn2_step(B, H, dk, dv, io, ge, qp, fp, vp, sp, op, st); });
    return wrap(std::move(o));
}

// fwd(q, f or z, beta or None, gated, v, h0, want_hT, o, hT, workspace, layout, chunk, flag)
PyObject* fwd(Args a, Py_ssize_t n)
{
    check_count(n, 13);
    const at::Tensor& q = tensor(a[0]); const at::Tensor& f = tensor(a[1]); const at::Tensor* beta = maybe_tensor(a[2]);
    const bool gated = to_bool(a[3]);
    const at::Tensor& v = tensor(a[4]); const at::Tensor* h0 = maybe_tensor(a[5]);
    const hgrn2_shape s = equal_shape(q, v, f, to_int(a[11]), to_int(a[10]), maybe_tensor(a[12]));
    if (gated) require(beta && beta->scalar_type() == at::kFloat && beta->dim() == 2 && beta->size(0) == s.H && beta->size(1) == s.dk, "beta: fp32 [H, dk]");
    else require(v.scalar_type() == q.scalar_type() && f.sizes() == q.sizes(), "q, f, v do not fit together");
    at::TensorBase o = given_or_like(maybe_tensor(a[7]), v);
    at::TensorBase hT = state_or_none(maybe_tensor(a[8]), to_bool(a[6]), s, q);
    at::TensorBase ws = workspace(maybe_tensor(a[9]), hgrn2_fwd_workspace_bytes(&s), q);
    const void *qp = ptr(q), *fp = ptr(f), *vp = ptr(v);
    const float *bp = fptr(beta), *hp = fptr(h0);
    void *op = ptr(o), *wp = ptr(ws), *st = stream();
    float* tp = out_fptr(hT);
    const size_t wb = (size_t)ws.numel();
    if (gated) enqueue("hgrn2_fwd_gated", [&] { return hgrn2_fwd_gated(&s, qp, fp, bp, vp, hp, op, tp, wp, wb, st); });
    else enqueue("hgrn2_fwd", [&] { return hgrn2_fwd(&s, qp, fp, vp, hp, op, tp, wp, wb, st); });
    return tuple_of(std::move(o), std::move(hT));
}

// fwd_saving(q, f, beta or None, v, h0, want_hT, o, hT, saved_states, workspace, layout, chunk, flag)
PyObject* fwd_saving(Args a, Py_ssize_t n)
{
    check_count(n, 13);
    const at::Tensor& q = tensor(a[0]); const at::Tensor& f = tensor(a[1]); const at::Tensor* beta = maybe_tensor(a[2]);
    const at::Tensor& v = tensor(a[3]); const at::Tensor* h0 = maybe_tensor(a[4]);
    const hgrn2_shape s = equal_shape(q, v, f, to_int(a[11]), to_int(a[10]), maybe_tensor(a[12]));
    at::TensorBase o = given_or_like(maybe_tensor(a[6]), v);
    at::TensorBase hT = state_or_none(maybe_tensor(a[7]), to_bool(a[5]), s, q);
    const at::Tensor* kept = maybe_tensor(a[8]);
    at::TensorBase saved = workspace(kept, kept ? 0 : hgrn2_saved_states_bytes(&s), q);
    at::TensorBase ws = workspace(maybe_tensor(a[9]), hgrn2_fwd_workspace_bytes(&s), q);
    const void *qp = ptr(q), *fp = ptr(f), *vp = ptr(v);
    const float *bp = fptr(beta), *hp = fptr(h0);
    void *op = ptr(o), *wp = ptr(ws), *sp = ptr(saved), *st = stream();
    float* tp = out_fptr(hT);
    const size_t wb = (size_t)ws.numel(), sb = (size_t)saved.numel();
    enqueue("hgrn2_fwd_saving", [&] { return hgrn2_fwd_saving(&s, qp, fp, bp, vp, hp, op, tp, sp, sb, wp, wb, st); });
    return tuple_of(std::move(o), std::move(hT), std::move(saved));
}

// bwd(kind, q, f, beta or None, v, h0 or saved_states, grad_o, grad_hT, want_grad_h0, grad_q, grad_f, grad_beta, grad_v,
//     grad_h0, workspace, layout, chunk, flag); kind: 0 hgrn2_bwd, 1 hgrn2_bwd_gated, 2 hgrn2_bwd_saved
PyObject* bwd(Args a, Py_ssize_t n)
{
    check_count(n, 18);
    const int kind = to_int(a[0]);
    const at::Tensor& q = tensor(a[1]); const at::Tensor& f = tensor(a[2]); const at::Tensor* beta = maybe_tensor(a[3]);
    const at::Tensor& v = tensor(a[4]); const at::Tensor* start = maybe_tensor(a[5]);
    const at::Tensor& go = tensor(a[6]); const at::Tensor* ghT = maybe_tensor(a[7]);
    const hgrn2_shape s = equal_shape(q, v, f, to_int(a[16]), to_int(a[15]), maybe_tensor(a[17]));
    at::TensorBase gq = given_or_like(maybe_tensor(a[9]), q), gf = given_or_like(maybe_tensor(a[10]), q);
    at::TensorBase gv = given_or_like(maybe_tensor(a[12]), v), gb;
    if (kind == 1 && !beta) fail(PyExc_TypeError, "beta is required");
    if (beta) gb = given_or_like(maybe_tensor(a[11]), *beta);
    at::TensorBase gh0 = state_or_none(maybe_tensor(a[13]), to_bool(a[8]), s, q);
    const size_t need = kind == 0 ? hgrn2_bwd_workspace_bytes(&s) : kind == 1 ? hgrn2_bwd_gated_workspace_bytes(&s)
                                  : hgrn2_bwd_saved_workspace_bytes(&s, beta ? 1 : 0);
    at::TensorBase ws = workspace(maybe_tensor(a[14]), need, q);
    const void *qp = ptr(q), *fp = ptr(f), *vp = ptr(v), *gop = ptr(go);
    const float *bp = fptr(beta), *gtp = fptr(ghT);
    void *gqp = ptr(gq), *gfp = ptr(gf), *gvp = ptr(gv), *wp = ptr(ws), *st = stream();
    float *gbp = out_fptr(gb), *ghp = out_fptr(gh0);
    const size_t wb = (size_t)ws.numel();
    if (kind == 2) {
        if (!start) fail(PyExc_TypeError, "saved_states is required");
        const void* sp = ptr(start);
        const size_t sb = (size_t)start->numel();
        enqueue("hgrn2_bwd_saved", [&] { return hgrn2_bwd_saved(&s, qp, fp, bp, vp, sp, sb, gop, gtp, gqp, gfp, gbp, gvp, ghp, wp, wb, st); });
    } else if (kind == 1) {
        const float* hp = fptr(start);
        enqueue("hgrn2_bwd_gated", [&] { return hgrn2_bwd_gated(&s, qp, fp, bp, vp, hp, gop, gtp, gqp, gfp, gbp, gvp, ghp, wp, wb, st); });
    } else {
        const float* hp = fptr(start);
        enqueue("hgrn2_bwd", [&] { return hgrn2_bwd(&s, qp, fp, vp, hp, gop, gtp, gqp, gfp, gvp, ghp, wp, wb, st); });
    }
    if (kind == 1) return tuple_of(std::move(gq), std::move(gf), std::move(gb), std::move(gv), std::move(gh0));
    if (beta) return tuple_of(std::move(gq), std::move(gf), std::move(gv), std::move(gh0), std::move(gb));
    return tuple_of(std::move(gq), std::move(gf), std::move(gv), std::move(gh0));
}

// fwd_varlen(q, f, beta or None, v, cu_seqlens, h0, want_hT, o, hT, saved_states or None, workspace, chunk, flag)
PyObject* fwd_varlen(Args a, Py_ssize_t n)
{
    check_count(n, 13);
    const at::Tensor& q = tensor(a[0]); const at::Tensor& f = tensor(a[1]); const at::Tensor* beta = maybe_tensor(a[2]);
    const at::Tensor& v = tensor(a[3]); const at::Tensor& cu = tensor(a[4]); const at::Tensor* h0 = maybe_tensor(a[5]);
    const hgrn2_shape s = packed_shape(q, v, f, cu, to_int(a[11]), maybe_tensor(a[12]));
    at::TensorBase o = given_or_like(maybe_tensor(a[7]), v);
    at::TensorBase hT = state_or_none(maybe_tensor(a[8]), to_bool(a[6]), s, q);
    const at::Tensor* saved = maybe_tensor(a[9]);
    at::TensorBase ws = workspace(maybe_tensor(a[10]), hgrn2_fwd_varlen_workspace_bytes(&s), q);
    const int32_t* cp = static_cast<const int32_t*>(ptr(cu));
    const void *qp = ptr(q), *fp = ptr(f), *vp = ptr(v);
    const float *bp = fptr(beta), *hp = fptr(h0);
    void *op = ptr(o), *wp = ptr(ws), *sp = ptr(saved), *st = stream();
    float* tp = out_fptr(hT);
    const size_t wb = (size_t)ws.numel(), sb = saved ? (size_t)saved->numel() : 0;
    if (saved) enqueue("hgrn2_fwd_varlen_saving", [&] { return hgrn2_fwd_varlen_saving(&s, cp, qp, fp, bp, vp, hp, op, tp, sp, sb, wp, wb, st); });
    else enqueue("hgrn2_fwd_varlen", [&] { return hgrn2_fwd_varlen(&s, cp, qp, fp, bp, vp, hp, op, tp, wp, wb, st); });
    return tuple_of(std::move(o), std::move(hT));
}

// bwd_varlen(q, f, beta or None, v, cu_seqlens, h0, saved_states or None, grad_o, grad_hT, want_grad_h0, grad_q, grad_f,
//            grad_v, workspace, chunk, flag)
PyObject* bwd_varlen(Args a, Py_ssize_t n)
{
    check_count(n, 16);
    const at::Tensor& q = tensor(a[0]); const at::Tensor& f = tensor(a[1]); const at::Tensor* beta = maybe_tensor(a[2]);
    const at::Tensor& v = tensor(a[3]); const at::Tensor& cu = tensor(a[4]); const at::Tensor* h0 = maybe_tensor(a[5]);
    const at::Tensor* saved = maybe_tensor(a[6]);
    const at::Tensor& go = tensor(a[7]); const at::Tensor* ghT = maybe_tensor(a[8]);
    const hgrn2_shape s = packed_shape(q, v, f, cu, to_int(a[14]), maybe_tensor(a[15]));
    at::TensorBase gq = given_or_like(maybe_tensor(a[10]), q), gf = given_or_like(maybe_tensor(a[11]), q);
    at::TensorBase gv = given_or_like(maybe_tensor(a[12]), v), gb, gh0;
    if (to_bool(a[9])) gh0 = state_tensor(s, q);
    if (beta) gb = fresh({s.H, s.dk}, at::kFloat, q);
    at::TensorBase ws = workspace(maybe_tensor(a[13]), hgrn2_bwd_varlen_workspace_bytes(&s), q);
    const int32_t* cp = static_cast<const int32_t*>(ptr(cu));
    const void *qp = ptr(q), *fp = ptr(f), *vp = ptr(v), *gop = ptr(go), *sp = ptr(saved);
    const float *bp = fptr(beta), *hp = fptr(h0), *gtp = fptr(ghT);
    void *gqp = ptr(gq), *gfp = ptr(gf), *gvp = ptr(gv), *wp = ptr(ws), *st = stream();
    float *gbp = out_fptr(gb), *ghp = out_fptr(gh0);
    const size_t wb = (size_t)ws.numel(), sb = saved ? (size_t)saved->numel() : 0;
    if (saved)
        enqueue("hgrn2_bwd_varlen_saved", [&] { return hgrn2_bwd_varlen_saved(&s, cp, qp, fp, bp, vp, hp, sp, sb, gop, gtp, gqp, gfp, gbp, gvp, ghp, wp, wb, st); });
    else
        enqueue("hgrn2_bwd_varlen", [&] { return hgrn2_bwd_varlen(&s, cp, qp, fp, bp, vp, hp, gop, gtp, gqp, gfp, gbp, gvp, ghp, wp, wb, st); });
    if (beta) return tuple_of(std::move(gq), std::move(gf), std::move(gv), std::move(gh0), std::move(gb));
    return tuple_of(std::move(gq), std::move(gf), std::move(gv), std::move(gh0));
}

// hgrn1_fwd(f, i, o, None, h0, ...); hgrn1_fwd_act(zf, zi, zo, beta, h0, want_hN, y, hN, workspace)
template <bool ACT> PyObject* h1_fwd(Args a, Py_ssize_t n)
{
    check_count(n, 9);
    const at::Tensor& f = tensor(a[0]); const at::Tensor& i = tensor(a[1]); const at::Tensor& o = tensor(a[2]);
    const at::Tensor* beta = maybe_tensor(a[3]); const at::Tensor* h0 = maybe_tensor(a[4]);
    if (i.dim() != 3) fail(PyExc_ValueError, "f, i, o must be 3-dimensional");
    const int32_t B = (int32_t)i.size(0), N = (int32_t)i.size(1), d = (int32_t)i.size(2);
    if (ACT) require(beta && i.sizes() == f.sizes() && o.sizes() == f.sizes() && beta->scalar_type() == at::kFloat && beta->numel() == d,
                      "zf, zi, zo, beta do not fit together");
    at::TensorBase y = given_or_like(maybe_tensor(a[6]), i), hN;
    if (const at::Tensor* given = maybe_tensor(a[7])) hN = *given;
    else if (to_bool(a[5])) hN = fresh({B, d}, at::kFloat, i);
    at::TensorBase ws = workspace(maybe_tensor(a[8]), hgrn1_workspace_bytes(B, N, d), i);
    const int32_t io = dtype_of(i), ge = dtype_of(f);
    const void *fp = ptr(f), *ip = ptr(i), *op = ptr(o);
    const float *bp = fptr(beta), *hp = fptr(h0);
    void *yp = ptr(y), *wp = ptr(ws), *st = stream();
    float* np = out_fptr(hN);
    const size_t wb = (size_t)ws.numel();
    if (ACT) enqueue("hgrn1_fwd_act", [&] { return hgrn1_fwd_act(B, N, d, io, ge, fp, ip, op, bp, hp, yp, np, wp, wb, st); });
    else enqueue("hgrn1_fwd", [&] { return hgrn1_fwd(B, N, d, io, ge, fp, ip, op, hp, yp, np, wp, wb, st); });
    return tuple_of(std::move(y), std::move(hN));
}

// hgrn1_bwd(f, i, o, None, grad_y, ...); hgrn1_bwd_act(zf, zi, zo, beta, grad_y, h0, grad_hN, want_grad_h0, workspace, saved)
template <bool ACT> PyObject* h1_bwd(Args a, Py_ssize_t n)
{
    check_count(n, 10);
    const at::Tensor& f = tensor(a[0]); const at::Tensor& i = tensor(a[1]); const at::Tensor& o = tensor(a[2]);
    const at::Tensor* beta = maybe_tensor(a[3]); const at::Tensor& gy = tensor(a[4]);
    const at::Tensor* h0 = maybe_tensor(a[5]); const at::Tensor* ghN = maybe_tensor(a[6]); const at::Tensor* given_ws = maybe_tensor(a[8]);
    const bool saved = to_bool(a[9]);
    require(given_ws || !saved, "saved=True needs the forward call's workspace");
    if (i.dim() != 3) fail(PyExc_ValueError, "f, i, o must be 3-dimensional");
    const int32_t B = (int32_t)i.size(0), N = (int32_t)i.size(1), d = (int32_t)i.size(2);
    at::TensorBase gf = fresh_like(i), gi = fresh_like(i), go = fresh_like(i), gb, gh0;
    if (ACT) {
        require(beta != nullptr, "beta: fp32 [d]");
        gb = fresh({d}, at::kFloat, i);
    }
    if (to_bool(a[7])) gh0 = fresh({B, d}, at::kFloat, i);
    at::TensorBase ws = workspace(given_ws, hgrn1_workspace_bytes(B, N, d), i);
    const int32_t io = dtype_of(i), ge = dtype_of(f);
    const void *fp = ptr(f), *ip = ptr(i), *op = ptr(o), *gyp = ptr(gy);
    const float *bp = fptr(beta), *hp = fptr(h0), *gnp = fptr(ghN);
    void *gfp = ptr(gf), *gip = ptr(gi), *gop = ptr(go), *wp = ptr(ws), *st = stream();
    float *gbp = out_fptr(gb), *ghp = out_fptr(gh0);
    const size_t wb = (size_t)ws.numel();
    if (ACT) {
        enqueue(saved ? "hgrn1_bwd_act_saved" : "hgrn1_bwd_act", [&] {
            return (saved ? hgrn1_bwd_act_saved : hgrn1_bwd_act)(B, N, d, io, ge, fp, ip, op, bp, hp, gyp, gnp, gfp, gip, gop, gbp, ghp, wp, wb, st);
        });
        return tuple_of(std::move(gf), std::move(gi), std::move(go), std::move(gb), std::move(gh0));
    }
    enqueue(saved ? "hgrn1_bwd_saved" : "hgrn1_bwd", [&] {
        return (saved ? hgrn1_bwd_saved : hgrn1_bwd)(B, N, d, io, ge, fp, ip, op, hp, gyp, gnp, gfp, gip, gop, ghp, wp, wb, st);
    });
    return tuple_of(std::move(gf), std::move(gi), std::move(go), std::move(gh0));
}

// proj_fwd(x, w3, b3, keep_av, z, v, q, av)
PyObject* proj_fwd(Args a, Py_ssize_t n)
{
    check_count(n, 8);
    const at::Tensor& x = tensor(a[0]); const at::Tensor& w3 = tensor(a[1]); const at::Tensor& b3 = tensor(a[2]);
    const int64_t d = x.size(-1);
    const int32_t M = d ? (int32_t)(x.numel() / d) : 0;
    require(w3.dim() == 2 && w3.size(0) == 3 * d && w3.size(1) == d && w3.scalar_type() == at::kBFloat16 && x.scalar_type() == at::kBFloat16,
            "x: bf16 [..., d], w3: bf16 [3d, d]");
    require(b3.scalar_type() == at::kFloat && b3.numel() == 3 * d, "b3: fp32 [3d]");
    at::TensorBase z = given_or_like(maybe_tensor(a[4]), x), v = given_or_like(maybe_tensor(a[5]), x), q = given_or_like(maybe_tensor(a[6]), x), av;
    if (const at::Tensor* given = maybe_tensor(a[7])) av = *given;
    else if (to_bool(a[3])) av = fresh_like(x);
    const void *xp = ptr(x), *wp = ptr(w3);
    const float* bp = static_cast<const float*>(ptr(b3));
    void *zp = ptr(z), *vp = ptr(v), *qp = ptr(q), *ap = out_ptr(av), *st = stream();
    enqueue("hgru2_proj_fwd", [&] { return hgru2_proj_fwd(M, (int32_t)d, xp, wp, bp, zp, vp, qp, ap, st); });
    return tuple_of(std::move(z), std::move(v), std::move(q), std::move(av));
}

// proj_bwd(x, w3, q, av, grad_z, grad_v, grad_q, workspace, grad_x, grad_w3, grad_b3)
PyObject* proj_bwd(Args a, Py_ssize_t n)
{
    check_count(n, 11);
    const at::Tensor& x = tensor(a[0]); const at::Tensor& w3 = tensor(a[1]); const at::Tensor& q = tensor(a[2]); const at::Tensor& av = tensor(a[3]);
    const at::Tensor& gz = tensor(a[4]); const at::Tensor& gv = tensor(a[5]); const at::Tensor& gq = tensor(a[6]);
    const int64_t d = x.size(-1);
    const int32_t M = d ? (int32_t)(x.numel() / d) : 0;
    at::TensorBase gx = given_or_like(maybe_tensor(a[8]), x), gw, gb;
    if (const at::Tensor* given = maybe_tensor(a[9])) gw = *given;
    else gw = fresh({3 * d, d}, at::kFloat, x);
    if (const at::Tensor* given = maybe_tensor(a[10])) gb = *given;
    else gb = fresh({3 * d}, at::kFloat, x);
    at::TensorBase ws = workspace(maybe_tensor(a[7]), hgru2_proj_bwd_workspace_bytes(M, (int32_t)d), x);
    const void *xp = ptr(x), *w3p = ptr(w3), *qp = ptr(q), *avp = ptr(av), *gzp = ptr(gz), *gvp = ptr(gv), *gqp = ptr(gq);
    void *gxp = ptr(gx), *wp = ptr(ws), *st = stream();
    float *gwp = out_fptr(gw), *gbp = out_fptr(gb);
    const size_t wb = (size_t)ws.numel();
    enqueue("hgru2_proj_bwd", [&] { return hgru2_proj_bwd(M, (int32_t)d, xp, w3p, qp, avp, gzp, gvp, gqp, gxp, gwp, gbp, wp, wb, st); });
    return tuple_of(std::move(gx), std::move(gw), std::move(gb));
}

// Exceptions stop here: a Python one is already set, a C++ one (the allocator's) becomes a RuntimeError,
// or torch's out-of-memory error where that is what it is.
template <PyObject* (*F)(Args, Py_ssize_t)> PyObject* entry(PyObject*, Args args, Py_ssize_t n)
{
    try {
        return F(args, n);
    } catch (const PyFail&) {
    } catch (const c10::OutOfMemoryError& e) {
        PyObject* cls = nullptr;
        if (PyObject* torch = PyImport_ImportModule("torch")) {
            cls = PyObject_GetAttrString(torch, "OutOfMemoryError");
            Py_DECREF(torch);
        }
        PyErr_SetString(cls ? cls : PyExc_MemoryError, e.what_without_backtrace());
        Py_XDECREF(cls);
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
    }
    return nullptr;
}

PyObject* set_error(PyObject*, PyObject* cls)
{
    Py_INCREF(cls);
    Py_XSETREF(hgrn2_error, cls);
    Py_RETURN_NONE;
}

#define HGRN2_ENTRY(name, fn) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&entry<fn>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    HGRN2_ENTRY("step", step<false>), HGRN2_ENTRY("step_gated", step<true>), HGRN2_ENTRY("fwd", fwd), HGRN2_ENTRY("fwd_saving", fwd_saving), HGRN2_ENTRY("bwd", bwd),
    HGRN2_ENTRY("fwd_varlen", fwd_varlen), HGRN2_ENTRY("bwd_varlen", bwd_varlen), HGRN2_ENTRY("hgrn1_fwd", h1_fwd<false>),
    HGRN2_ENTRY("hgrn1_fwd_act", h1_fwd<true>), HGRN2_ENTRY("hgrn1_bwd", h1_bwd<false>), HGRN2_ENTRY("hgrn1_bwd_act", h1_bwd<true>),
    HGRN2_ENTRY("proj_fwd", proj_fwd), HGRN2_ENTRY("proj_bwd", proj_bwd),
    {"set_error", set_error, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}   // namespace

PyMODINIT_FUNC PyInit__host(void) { return PyModule_Create(&module); }
