// Native part of the Python binding: argument checks, output and workspace allocation and
// the C ABI call of the filter layer's entry points (include/kla.h), for
// paper_2602_10743_amd/__init__.py.
//
// A training step of a few sequences is bound by the host: through ctypes and torch.empty the
// forward took 21 us and the backward 33 us of it, more than their kernels.  Functions return the
// output tensors, or the status code when the library refuses the call.  Past the checks they give
// up the interpreter lock, as ctypes does: allocations and a full launch queue can block, and under
// KLA_CHECK=1 the library waits for the stream.
#include <array>
#include <string>

#include <c10/hip/HIPStream.h>
#include <torch/extension.h>

#include "kla.h"

namespace py = pybind11;
using at::Tensor;
using Opt = c10::optional<Tensor>;

namespace {

const char* kNames[6] = {"q", "k", "v", "a", "p", "r"};

[[noreturn]] void value_error(const std::string& s) { throw py::value_error(s); }

std::string shape_str(at::IntArrayRef s) {
    std::string o = "(";
    for (size_t i = 0; i < s.size(); ++i) o += (i ? ", " : "") + std::to_string(s[i]);
    return o + (s.size() == 1 ? ",)" : ")");
}

int dtype_of(const Tensor& q) {
    if (q.scalar_type() == at::kFloat) return KLA_F32;
    if (q.scalar_type() == at::kBFloat16) return KLA_BF16;
    throw py::type_error("unsupported dtype " + std::string(py::str(py::cast(q).attr("dtype"))) +
                         "; use float32 or bfloat16");
}

void* ptr(const Tensor& t) { return t.data_ptr(); }
void* ptr(const Opt& t) { return t ? t->data_ptr() : nullptr; }
float* fptr(const Opt& t) { return static_cast<float*>(ptr(t)); }

hipStream_t stream_of(const Tensor& t) { return c10::hip::getCurrentHIPStream(t.device().index()).stream(); }

// q [B, T, H, dk] and the other per-token tensors (a, p absent with OU gates)
kla_desc check_inputs(const Tensor& q, const Tensor& k, const Tensor& v, const Tensor* a, const Tensor* p,
                      const Tensor& r) {
    if (!q.is_cuda()) value_error("KLA tensors must live on a GPU; the layer has no CPU path");
    const int dt = dtype_of(q);
    if (q.dim() != 4) value_error("q must be [B, T, H, dk]");
    const int64_t B = q.size(0), T = q.size(1), H = q.size(2), dk = q.size(3), dv = v.size(-1);
    const std::array<int64_t, 4> ks{B, T, H, dk}, vs{B, T, H, dv};
    const std::array<int64_t, 3> rs{B, T, H};
    const Tensor* t[6] = {&q, &k, &v, a, p, &r};
    for (int i : {1, 3, 4, 2, 5}) {
        if (!t[i]) continue;
        const at::IntArrayRef want = i == 2 ? at::IntArrayRef(vs) : i == 5 ? at::IntArrayRef(rs) : at::IntArrayRef(ks);
        if (t[i]->sizes() != want)
            value_error(std::string(kNames[i]) + " has shape " + shape_str(t[i]->sizes()) + ", expected " + shape_str(want));
        if (t[i]->scalar_type() != q.scalar_type() || t[i]->device() != q.device())
            value_error(std::string(kNames[i]) + " must share q's dtype and device");
    }
    for (int i = 0; i < 6; ++i)
        if (t[i] && !t[i]->is_contiguous()) value_error(std::string(kNames[i]) + " must be contiguous");
    return kla_desc{(int32_t)B, (int32_t)T, (int32_t)H, (int32_t)dk, (int32_t)dv, (kla_dtype)dt};
}

void check_f32(const Opt& t, at::IntArrayRef shape, const Tensor& q, const char* name) {
    if (!t) return;
    if (t->scalar_type() != at::kFloat || t->sizes() != shape || t->device() != q.device() || !t->is_contiguous())
        value_error(std::string(name) + " must be a contiguous float32 tensor of shape " + shape_str(shape) + " on " +
                    q.device().str());
}

void check_belief(const kla_desc& d, const Opt& lam, const Opt& eta, const Tensor& q, const char* ln, const char* en) {
    check_f32(lam, {d.B, d.H, d.dk}, q, ln);
    check_f32(eta, {d.B, d.H, d.dk, d.dv}, q, en);
}

void check_ou(const Opt& a, const Opt& p, const Opt& delta, int64_t H, int64_t dk, const Tensor& q) {
    check_f32(a, {H, dk}, q, "a");
    check_f32(p, {H, dk}, q, "p");
    check_f32(delta, {H, dk}, q, "delta");
}

// a per-token gate tensor, which has to be there (none with OU gates)
const Tensor* per_token(const Opt& t, bool ou, const char* name) {
    if (ou) return nullptr;
    if (!t) throw py::type_error(std::string(name) + " must be a tensor");
    return &*t;
}

Tensor bytes(size_t n, const Tensor& q) {
    return at::empty({(int64_t)(n > 1 ? n : 1)}, q.options().dtype(at::kByte));
}

py::object obj(const Opt& t) { return t ? py::cast(*t) : py::none(); }

// (y, yvar, lamT, etaT, saved) or a status.  ou: OU gates, a, p, delta [H, dk] fp32 (the library
// refuses the call when one is absent).
py::object forward(const Tensor& q, const Tensor& k, const Tensor& v, const Opt& a, const Opt& p, const Opt& delta,
                   const Tensor& r, const Opt& lam0, const Opt& eta0, const Opt& y_in, bool want_var, bool want_state,
                   bool save, bool ou) {
    const kla_desc d = check_inputs(q, k, v, per_token(a, ou, "a"), per_token(p, ou, "p"), r);
    if (ou) check_ou(a, p, delta, d.H, d.dk, q);
    check_belief(d, lam0, eta0, q, "lam0", "eta0");
    Tensor y;
    Opt yvar, lamT, etaT, saved;
    kla_status st;
    {
        py::gil_scoped_release unlocked;
        const auto f32 = q.options().dtype(at::kFloat);
        y = y_in ? *y_in : at::empty({d.B, d.T, d.H, d.dv}, q.options());
        if (want_var) yvar = at::empty({d.B, d.T, d.H}, f32);
        if (want_state) {
            lamT = at::empty({d.B, d.H, d.dk}, f32);
            etaT = at::empty({d.B, d.H, d.dk, d.dv}, f32);
        }
        const size_t ns = save ? kla_saved_bytes(&d) : 0, nw = kla_forward_workspace(&d);
        if (ns) saved = bytes(ns, q);
        const Tensor ws = bytes(nw, q);
        st = ou ? kla_forward_ou(&d, ptr(q), ptr(k), ptr(v), (const float*)ptr(a), (const float*)ptr(p), fptr(delta),
                                 ptr(r), fptr(lam0), fptr(eta0), ptr(y), fptr(yvar), fptr(lamT), fptr(etaT), ptr(saved),
                                 ptr(ws), nw, stream_of(q))
                : kla_forward(&d, ptr(q), ptr(k), ptr(v), ptr(a), ptr(p), ptr(r), fptr(lam0), fptr(eta0), ptr(y),
                              fptr(yvar), fptr(lamT), fptr(etaT), ptr(saved), ptr(ws), nw, stream_of(q));
    }
    if (st != KLA_OK) return py::int_((int)st);
    return py::make_tuple(y, obj(yvar), obj(lamT), obj(etaT), obj(saved));
}

// (dq, dk, dv, da, dp, dr, dlam0, deta0[, ddelta]) or a status
py::object backward(const Tensor& q, const Tensor& k, const Tensor& v, const Opt& a, const Opt& p, const Opt& delta,
                    const Tensor& r, const Opt& lam0, const Opt& eta0, const Tensor& dy, const Opt& dlamT,
                    const Opt& detaT, const Opt& saved, bool want_init, const Opt& dyvar, bool noalloc, bool ou) {
    const kla_desc d = check_inputs(q, k, v, per_token(a, ou, "a"), per_token(p, ou, "p"), r);
    if (ou) check_ou(a, p, delta, d.H, d.dk, q);
    check_belief(d, lam0, eta0, q, "lam0", "eta0");
    check_belief(d, dlamT, detaT, q, "dlamT", "detaT");
    check_f32(dyvar, {d.B, d.T, d.H}, q, "dyvar");
    if (dy.sizes() != at::IntArrayRef({d.B, d.T, d.H, d.dv}) || dy.scalar_type() != q.scalar_type() || !dy.is_contiguous())
        value_error("dy must be a contiguous [B, T, H, dv] tensor in the input dtype");
    Tensor dq, dk, dv, da, dp, dr;
    Opt ddelta, dlam0, deta0;
    kla_status st;
    {
        py::gil_scoped_release unlocked;
        const auto f32 = q.options().dtype(at::kFloat);
        dq = at::empty_like(q), dk = at::empty_like(k), dv = at::empty_like(v), dr = at::empty_like(r);
        da = ou ? at::empty({d.H, d.dk}, f32) : at::empty_like(*a);
        dp = ou ? at::empty({d.H, d.dk}, f32) : at::empty_like(*p);
        if (ou) ddelta = at::empty({d.H, d.dk}, f32);
        if (want_init) {
            dlam0 = at::empty({d.B, d.H, d.dk}, f32);
            deta0 = at::empty({d.B, d.H, d.dk, d.dv}, f32);
        }
        if (noalloc) {
            st = kla_backward_noalloc(&d, ptr(q), ptr(k), ptr(v), ptr(a), ptr(p), ptr(r), fptr(lam0), fptr(eta0), ptr(saved),
                                      ptr(dy), fptr(dyvar), fptr(dlamT), fptr(detaT), ptr(dq), ptr(dk), ptr(dv), ptr(da),
                                      ptr(dp), ptr(dr), fptr(dlam0), fptr(deta0), stream_of(q));
        } else if (ou) {
            const size_t nw = kla_backward_ou_workspace(&d, saved.has_value());
            const Tensor ws = bytes(nw, q);
            st = kla_backward_ou(&d, ptr(q), ptr(k), ptr(v), (const float*)ptr(a), (const float*)ptr(p), fptr(delta), ptr(r),
                                 fptr(lam0), fptr(eta0), ptr(saved), ptr(dy), fptr(dyvar), fptr(dlamT), fptr(detaT), ptr(dq),
                                 ptr(dk), ptr(dv), (float*)ptr(da), (float*)ptr(dp), fptr(ddelta), ptr(dr), fptr(dlam0),
                                 fptr(deta0), ptr(ws), nw, stream_of(q));
        } else {
            const size_t nw = kla_backward_workspace(&d, saved.has_value());
            const Tensor ws = bytes(nw, q);
            st = kla_backward(&d, ptr(q), ptr(k), ptr(v), ptr(a), ptr(p), ptr(r), fptr(lam0), fptr(eta0), ptr(saved), ptr(dy),
                              fptr(dyvar), fptr(dlamT), fptr(detaT), ptr(dq), ptr(dk), ptr(dv), ptr(da), ptr(dp), ptr(dr),
                              fptr(dlam0), fptr(deta0), ptr(ws), nw, stream_of(q));
        }
    }
    if (st != KLA_OK) return py::int_((int)st);
    if (ou) return py::make_tuple(dq, dk, dv, da, dp, dr, obj(dlam0), obj(deta0), *ddelta);
    return py::make_tuple(dq, dk, dv, da, dp, dr, obj(dlam0), obj(deta0));
}

// (y, yvar) or a status; lam, eta updated in place
py::object decode_step(const Tensor& q, const Tensor& k, const Tensor& v, const Opt& a, const Opt& p,
                       const Opt& delta, const Tensor& r, const Opt& lam, const Opt& eta, const Opt& y_in,
                       bool want_var, bool ou) {
    if (!q.is_cuda() || (q.scalar_type() != at::kFloat && q.scalar_type() != at::kBFloat16))
        value_error("decode inputs must be fp32/bf16 GPU tensors");
    if (q.dim() != 3) value_error("q must be [S, H, dk]");
    const int64_t S = q.size(0), H = q.size(1), dk = q.size(2), dv = v.size(-1);
    const std::array<int64_t, 3> ks{S, H, dk}, vs{S, H, dv};
    const std::array<int64_t, 2> rs{S, H};
    const Tensor* t[6] = {&q, &k, &v, per_token(a, ou, "a"), per_token(p, ou, "p"), &r};
    for (int i : {1, 3, 4, 2, 5}) {
        if (!t[i]) continue;
        const at::IntArrayRef want = i == 2 ? at::IntArrayRef(vs) : i == 5 ? at::IntArrayRef(rs) : at::IntArrayRef(ks);
        if (t[i]->sizes() != want || t[i]->scalar_type() != q.scalar_type() || !t[i]->is_contiguous())
            value_error(std::string(kNames[i]) + " must be a contiguous " + shape_str(want) + " tensor in q's dtype");
    }
    if (ou) check_ou(a, p, delta, H, dk, q);
    check_f32(lam, {S, H, dk}, q, "lam");
    check_f32(eta, {S, H, dk, dv}, q, "eta");
    const kla_dtype dt = (kla_dtype)dtype_of(q);
    Tensor y;
    Opt yvar;
    kla_status st;
    {
        py::gil_scoped_release unlocked;
        y = y_in ? *y_in : at::empty({S, H, dv}, q.options());
        if (want_var) yvar = at::empty({S, H}, q.options().dtype(at::kFloat));
        st = ou ? kla_decode_step_ou(S, H, dk, dv, dt, ptr(q), ptr(k), ptr(v), (const float*)ptr(a),
                                     (const float*)ptr(p), fptr(delta), ptr(r), fptr(lam), fptr(eta),
                                     ptr(y), fptr(yvar), stream_of(q))
                : kla_decode_step(S, H, dk, dv, dt, ptr(q), ptr(k), ptr(v), ptr(a), ptr(p), ptr(r), fptr(lam),
                                  fptr(eta), ptr(y), fptr(yvar), stream_of(q));
    }
    if (st != KLA_OK) return py::int_((int)st);
    return py::make_tuple(y, obj(yvar));
}

}  // namespace

PYBIND11_MODULE(_kla_torch, m) {
    m.def("forward", &forward);
    m.def("backward", &backward);
    m.def("decode_step", &decode_step);
}
