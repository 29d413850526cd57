// Pattern and forward pass as one call: the launches of spa2_mask and spa2_fwd in sequence, with what one of them can do
// for the next.  On small layers the pooling pass zeroes the arrival counters of split rows, and the sizes alone say how
// rows are cut, so that no plan is launched: sampling on two heads of 1,000 tokens 21.2 -> 17.6 us a pass.
#include "spa2_check.h"
#include "spa2_internal.h"

using namespace spa2;

namespace {
// Workspace: the forward section, whose pool is free until the forward kernel runs: the pooled means lie there.
SplitPlan fwd_section(const Dims& m, void* ws, size_t bytes) {
  return with_stretches(split_layout(ws, bytes, (int64_t)m.B * m.H * m.Tm, m.Tn, fwd_slot_bytes(m)), m);
}
size_t fwd_bytes(const Dims& m) {
  return round256(split_ws_bytes((int64_t)m.B * m.H * m.Tm, m.Tn, fwd_slot_bytes(m)));
}
size_t pool_offset(const Dims& m) { return split_pool_offset((int64_t)m.B * m.H * m.Tm, m.Tn); }
}  // namespace

extern "C" {

size_t spa2_mask_fwd_workspace_bytes(const spa2_shape* shape) {
  if (check_shape(shape) != SPA2_OK) return 0;
  const Dims m = make_dims(*shape);
  const size_t f = fwd_bytes(m), p = pool_offset(m) + mask_ws(m).total;
  return f > p ? f : p;
}

int spa2_mask_fwd(const void* q, const void* k, const void* v, const spa2_shape* shape, int32_t topk_blocks, float top_p,
                  float scale, spa2_pattern* out, void* o, void* o_res, float* lse, void* workspace, size_t workspace_bytes,
                  void* stream) {
  int rc = check_mask(q, k, shape, topk_blocks, top_p, scale, out);
  if (rc != SPA2_OK) return rc;
  rc = check_fwd(q, k, v, shape, out, scale, o, o_res, lse);
  if (rc != SPA2_OK) return rc;
  const Dims m = make_dims(*shape);
  if (!workspace || workspace_bytes < spa2_mask_fwd_workspace_bytes(shape)) return SPA2_ERR_WORKSPACE;
  if (!aligned16(workspace)) return SPA2_ERR_ALIGN;
  const int64_t units = (int64_t)m.B * m.H * m.Tm;
  const SplitPlan plan = with_fixed_parts(fwd_section(m, workspace, fwd_bytes(m)), units, m.Tn);
  char* means = (char*)workspace + pool_offset(m);
  const MaskWs w = mask_ws(m);
  if (launch_pool_zero(q, k, m, (float*)(means + w.qbar), (float*)(means + w.kbar), plan.arrive,
                       plan.fixed_len ? (int)units * plan.fixed_parts : 0, (hipStream_t)stream) != hipSuccess)
    return SPA2_ERR_LAUNCH;
  rc = spa2_mask_select(shape, topk_blocks, top_p, scale, out, nullptr, means, w.total, stream);
  if (rc != SPA2_OK) return rc;
  if (out->col_cnt) rc = spa2_mask_columns(shape, out, stream);
  if (rc != SPA2_OK) return rc;
  return launch_fwd(q, k, v, m, out->row_cnt, out->row_idx, out->row_order, scale, o, o_res, lse, plan,
                    (hipStream_t)stream) == hipSuccess ? SPA2_OK : SPA2_ERR_LAUNCH;
}

}  // extern "C"
