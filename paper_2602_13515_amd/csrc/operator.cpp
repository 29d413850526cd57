// The two differentiable operators in native code: block-sparse attention (pattern from q and k, forward, backward) and
// the velocity distillation loss, as autograd functions over the C ABI.  Same results, checks and errors as the Python
// functions in autograd.py and distill.py, which stay for the calls that this module does not take (a pattern asked for,
// overlapping backward kernels, tracing, function transforms, tensors that are not plain CUDA tensors).
//
// Why: the Python route cost more host time than the kernels take on small layers.  Two heads of 2,048 tokens, forward and
// backward: 82 us of kernels and the gaps between them, 226 us a pass, in which the backward pass waited for the
// interpreter lock twice.  Here a pass allocates one buffer for the pattern (six tensors before) and one scratch buffer for
// mask and forward, and the backward pass runs in the engine's thread without the interpreter: 90 us (82 with the
// kernels as they are now).  24 heads of 1,281 tokens 223 -> 133 us (116); sampling on 1,000 tokens, two heads 46 -> 28 us (17).
#include <c10/core/DeviceGuard.h>
#include <c10/hip/HIPStream.h>
#include <torch/extension.h>

#include "spa2.h"

namespace {

using at::Tensor;
using torch::autograd::AutogradContext;
using torch::autograd::Variable;
using torch::autograd::variable_list;

// A negative return code of the C ABI as the exception the Python binding raises for it.
void check(int code, const char* where) {
  if (code == SPA2_OK) return;
  py::gil_scoped_acquire gil;
  const py::object e = py::module_::import("paper_2602_13515_amd.binding").attr("Spa2Error")(code, where);
  PyErr_SetObject((PyObject*)Py_TYPE(e.ptr()), e.ptr());
  throw py::error_already_set();
}

void* stream_of(const Tensor& x) { return (void*)c10::hip::getCurrentHIPStream(x.device().index()).stream(); }

Tensor like(const Tensor& x) { return at::empty_strided(x.sizes(), x.strides(), x.options()); }

Tensor bytes(int64_t n, const Tensor& x) { return at::empty({n}, x.options().dtype(at::kByte)); }

// x with ref's strides (the kernels take one stride triple for all token tensors of a call).
Tensor match(const Tensor& x, const Tensor& ref) {
  if (x.strides() == ref.strides()) return x;
  Tensor y = like(ref);
  y.copy_(x);
  return y;
}

constexpr const char* ONE_LAYOUT = "all token tensors of one call share shape, strides, dtype and device";

void same_layout(const Tensor& ref, std::initializer_list<const Tensor*> others) {
  for (const Tensor* t : others)
    TORCH_CHECK_VALUE(t->sizes() == ref.sizes() && t->strides() == ref.strides() &&
                      t->scalar_type() == ref.scalar_type() && t->device() == ref.device(), ONE_LAYOUT);
}

void check_inputs(const Tensor& q, const Tensor& k, const Tensor& v) {
  const std::pair<const char*, const Tensor*> named[] = {{"q", &q}, {"k", &k}, {"v", &v}};
  for (const auto& [name, t] : named) {
    TORCH_CHECK_VALUE(t->is_cuda(), name, " must live on the GPU: the operator has no CPU path");
    TORCH_CHECK_VALUE(t->scalar_type() == at::kBFloat16 && t->dim() == 4, name, " must be a bf16 [B, H, N, d] view");
  }
  TORCH_CHECK_VALUE(k.sizes() == q.sizes() && v.sizes() == q.sizes(), "self-attention: q, k, v share one shape");
  TORCH_CHECK_VALUE(q.stride(3) == 1, "the head dimension must be contiguous");
  TORCH_CHECK_VALUE(k.device() == q.device() && v.device() == q.device(), ONE_LAYOUT);
}

// What saved-tensor hooks bring back is checked before a kernel gets its address.  (The sizes are those of the upstream
// gradient, which the engine has compared with the output's.)
void check_saved(const Tensor& q, const Tensor& lse, int64_t gpu) {
  TORCH_CHECK_VALUE(q.is_cuda() && q.device().index() == gpu && q.scalar_type() == at::kBFloat16 && q.dim() == 4 &&
                    q.stride(3) == 1, "saved token tensors come back as bf16 [B, H, N, d] views on their GPU, d contiguous");
  TORCH_CHECK_VALUE(lse.device() == q.device() && lse.scalar_type() == at::kFloat && lse.is_contiguous() &&
                    lse.numel() == q.size(0) * q.size(1) * q.size(2), "the log-sum-exp comes back as B * H * N contiguous fp32 numbers");
}

spa2_shape shape_of(const Tensor& q) {
  spa2_shape s;
  s.B = (int32_t)q.size(0); s.H = (int32_t)q.size(1); s.N = (int32_t)q.size(2); s.d = (int32_t)q.size(3);
  s.bq = SPA2_BQ; s.bkv = SPA2_BKV;
  s.sb = q.stride(0); s.sh = q.stride(1); s.sn = q.stride(2);
  return s;
}

// The arrays of a pattern of our own in one buffer.  The backward pass makes the column lists (spa2_bwd_rows).
struct PatternLayout {
  int64_t off[3] = {0, 0, 0}, total = 0;
  explicit PatternLayout(const spa2_shape& s) {
    const int64_t bh = (int64_t)s.B * s.H;
    const int64_t tm = ((int64_t)s.N + SPA2_BQ - 1) / SPA2_BQ, tn = ((int64_t)s.N + SPA2_BKV - 1) / SPA2_BKV;
    const int64_t size[3] = {bh * tm * tn, 4 * bh * tm, 4 * bh * tm * tn};
    for (int x = 0; x < 3; ++x) { off[x] = total; total += (size[x] + 255) & ~(int64_t)255; }
  }
  spa2_pattern in(const Tensor& buf) const {
    char* p = (char*)buf.data_ptr();
    spa2_pattern r = {};
    r.mask = (uint8_t*)(p + off[0]);
    r.row_cnt = (int32_t*)(p + off[1]); r.row_idx = (int32_t*)(p + off[2]);
    return r;
  }
};

// A caller's pattern: mask, row_cnt, row_idx, col_cnt, col_idx, row_order, col_order (undefined: not there).
spa2_pattern given_pattern(const std::vector<Tensor>& t) {
  auto at = [&](int x) -> void* { return t[x].defined() ? t[x].data_ptr() : nullptr; };
  spa2_pattern r;
  r.mask = (uint8_t*)at(0);
  r.row_cnt = (int32_t*)at(1); r.row_idx = (int32_t*)at(2);
  r.col_cnt = (int32_t*)at(3); r.col_idx = (int32_t*)at(4);
  r.row_order = (int32_t*)at(5); r.col_order = (int32_t*)at(6);
  return r;
}

struct Attention : torch::autograd::Function<Attention> {
  static Tensor forward(AutogradContext* ctx, const Tensor& q, const Tensor& k_in, const Tensor& v_in, double k_frac,
                        double top_p, double scale, bool training, const std::vector<Tensor>& given) {
    const c10::DeviceGuard device(q.device());
    const Tensor k = match(k_in, q), v = match(v_in, q);
    const spa2_shape s = shape_of(q);
    const bool build = given.empty();
    const PatternLayout layout(s);
    const Tensor buf = build ? bytes(layout.total, q) : Tensor();
    spa2_pattern pattern = build ? layout.in(buf) : given_pattern(given);
    // one scratch buffer for mask and forward; a log-sum-exp that nobody reads lies behind it
    const int64_t need = (int64_t)(build ? spa2_mask_fwd_workspace_bytes(&s) : spa2_fwd_workspace_bytes(&s));
    const int64_t lse_at = (need + 255) & ~(int64_t)255;
    const Tensor ws = bytes(training ? lse_at : lse_at + 4 * q.size(0) * q.size(1) * q.size(2), q);
    void* stream = stream_of(q);
    const int32_t tn = (int32_t)((q.size(2) + SPA2_BKV - 1) / SPA2_BKV);
    const Tensor o = like(q);
    Tensor o_res, lse;
    if (training) {
      o_res = like(q);
      lse = at::empty({q.size(0), q.size(1), q.size(2)}, q.options().dtype(at::kFloat));
    }
    float* lse_p = training ? (float*)lse.data_ptr() : (float*)((char*)ws.data_ptr() + lse_at);
    void* o_res_p = training ? o_res.data_ptr() : nullptr;
    if (build)
      check(spa2_mask_fwd(q.data_ptr(), k.data_ptr(), v.data_ptr(), &s, spa2_topk_blocks(k_frac, tn), (float)top_p,
                          (float)scale, &pattern, o.data_ptr(), o_res_p, lse_p, ws.data_ptr(), (size_t)need, stream),
            "spa2_mask_fwd");
    else
      check(spa2_fwd(q.data_ptr(), k.data_ptr(), v.data_ptr(), &s, &pattern, (float)scale, o.data_ptr(), o_res_p, lse_p,
                     ws.data_ptr(), (size_t)need, stream), "spa2_fwd");
    if (training) {
      ctx->save_for_backward({q, k, v, o, o_res, lse});
      ctx->saved_data["pattern"] = build ? std::vector<Tensor>{buf} : given;
      ctx->saved_data["scale"] = scale;
      ctx->saved_data["gpu"] = (int64_t)q.device().index();
    }
    return o;
  }

  static variable_list backward(AutogradContext* ctx, variable_list grads) {
    const variable_list saved = ctx->get_saved_variables();
    const Tensor &q = saved[0], &k = saved[1], &v = saved[2], &o = saved[3], &o_res = saved[4], &lse = saved[5];
    check_saved(q, lse, ctx->saved_data["gpu"].toInt());
    const c10::DeviceGuard device(q.device());
    const Tensor d_o = match(grads[0].to(at::kBFloat16), q);
    // (all of them, not d_o alone: saved-tensor hooks may bring a tensor back in another layout)
    same_layout(q, {&k, &v, &o, &o_res, &d_o});
    const spa2_shape s = shape_of(q);
    const std::vector<Tensor> kept = ctx->saved_data["pattern"].toTensorVector();
    const bool built = kept.size() == 1;
    const spa2_pattern pattern = built ? PatternLayout(s).in(kept[0]) : given_pattern(kept);
    const Tensor dq = like(q), dk = like(q), dv = like(q);
    const int64_t need = (int64_t)(built ? spa2_bwd_rows_workspace_bytes(&s) : spa2_bwd_workspace_bytes(&s));
    const Tensor ws = bytes(need, q);
    check((built ? spa2_bwd_rows : spa2_bwd)(q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(), o_res.data_ptr(),
                                             d_o.data_ptr(), (const float*)lse.data_ptr(), &s, &pattern,
                                             (float)ctx->saved_data["scale"].toDouble(), dq.data_ptr(), dk.data_ptr(),
                                             dv.data_ptr(), ws.data_ptr(), (size_t)need, stream_of(q)),
          built ? "spa2_bwd_rows" : "spa2_bwd");
    return {dq, dk, dv, Variable(), Variable(), Variable(), Variable(), Variable()};
  }
};

// given: a caller's pattern (see given_pattern), or none: it is built from q and k
Tensor attention(const Tensor& q, const Tensor& k, const Tensor& v, double k_frac, double top_p, double scale,
                 const std::vector<std::optional<Tensor>>& given) {
  check_inputs(q, k, v);
  // Without a backward pass to come (sampling) nobody reads the column lists or the output's residual.
  const bool training = at::GradMode::is_enabled() && (q.requires_grad() || k.requires_grad() || v.requires_grad());
  std::vector<Tensor> pattern;
  for (const auto& t : given) pattern.push_back(t.value_or(Tensor()));
  return Attention::apply(q, k, v, k_frac, top_p, scale, training, pattern);
}

// ------------------------------------------------------------------ velocity distillation loss
int32_t vd_type(const Tensor& x) { return x.scalar_type() == at::kBFloat16 ? 0 : 1; }

void vd_check(const Tensor& us, const Tensor& uf) {
  TORCH_CHECK_VALUE(us.is_cuda() && uf.is_cuda(), "spa2 runs on the GPU only: predictions must be CUDA tensors");
  TORCH_CHECK_VALUE((us.scalar_type() == at::kBFloat16 || us.scalar_type() == at::kFloat) &&
                    uf.scalar_type() == us.scalar_type(), "predictions are bfloat16 or float32, both of the same type");
  TORCH_CHECK_VALUE(us.sizes() == uf.sizes() && us.is_contiguous() && uf.is_contiguous() && us.device() == uf.device(),
                    "predictions are contiguous tensors of one shape");
}

// One pass for the loss, one for the gradient.  (Not spa2_vd_loss_and_grad: what the upstream derivative is, and whether a
// backward pass comes at all, is known only after the loss.  With it, 2 x 201 MB of fp32, us: upstream 1 172 -> 115, but upstream
// 0.5 171 -> 191 and the loss alone 74 -> 111, and a gradient that is multiplied afterwards is rounded once more.)
struct VelocityLoss : torch::autograd::Function<VelocityLoss> {
  static Tensor forward(AutogradContext* ctx, const Tensor& us, const Tensor& uf, double weight) {
    vd_check(us, uf);
    const c10::DeviceGuard device(us.device());
    const Tensor loss = at::empty({}, us.options().dtype(at::kDouble));
    const int64_t n = (int64_t)spa2_vd_loss_workspace_bytes();
    const Tensor ws = bytes(n, us);
    check(spa2_vd_loss(us.data_ptr(), uf.data_ptr(), us.numel(), vd_type(us), weight, (double*)loss.data_ptr(),
                       ws.data_ptr(), (size_t)n, stream_of(us)), "spa2_vd_loss");
    ctx->save_for_backward({us, uf});
    ctx->saved_data["weight"] = weight;
    return loss;
  }

  static variable_list backward(AutogradContext* ctx, variable_list grads) {
    const variable_list saved = ctx->get_saved_variables();
    const Tensor &us = saved[0], &uf = saved[1];
    vd_check(us, uf);
    const c10::DeviceGuard device(us.device());
    const Tensor upstream = grads[0].contiguous();
    TORCH_CHECK_VALUE(upstream.scalar_type() == at::kDouble && upstream.numel() == 1 && upstream.is_cuda(),
                      "upstream is a float64 CUDA tensor of one element");
    const Tensor grad = at::empty_like(us);
    check(spa2_vd_loss_grad(us.data_ptr(), uf.data_ptr(), us.numel(), vd_type(us), ctx->saved_data["weight"].toDouble(),
                            (const double*)upstream.data_ptr(), grad.data_ptr(), stream_of(us)), "spa2_vd_loss_grad");
    return {grad, Variable(), Variable()};
  }
};

Tensor velocity_loss(const Tensor& u_sparse, const Tensor& u_full, double weight) {
  return VelocityLoss::apply(u_sparse.contiguous(), u_full.detach().contiguous(), weight);
}

}  // namespace

PYBIND11_MODULE(TORCH_EXTENSION_NAME, m) {
  m.def("attention", &attention, py::call_guard<py::gil_scoped_release>());
  m.def("velocity_loss", &velocity_loss, py::call_guard<py::gil_scoped_release>());
}
