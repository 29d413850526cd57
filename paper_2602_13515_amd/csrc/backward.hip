// The backward pass of a pattern that came without column lists: these, the launch order of the key blocks and the plan of
// the dK/dV kernel are made by workgroups of the launches in front of it, the lists beside D, order and plan in the launch
// of dQ, which needs neither.  Against column lists and order as launches of the forward pass and dK/dV before dQ, us a
// training pass, before / after: 4 samples of 1281 tokens, 6 heads 111.2 / 107.6; 20,010 tokens, 6 heads, d = 64 296.4 / 291.4;
// 32,760 tokens, 12 heads 1919 / 1910; 2285 tokens, 24 heads, d = 64 131.6 / 128.6.
#include "spa2_check.h"
#include "spa2_internal.h"

using namespace spa2;

namespace {
// Workspace: that of spa2_bwd, then col_cnt, col_idx, col_order.
struct RowsWs { size_t cnt, idx, order, total; };
RowsWs rows_ws(const Dims& m) {
  const size_t cols = (size_t)m.B * m.H * m.Tn;
  RowsWs w;
  w.cnt = round256(bwd_ws(m).total);
  w.idx = w.cnt + round256(4 * cols);
  w.order = w.idx + round256(4 * cols * m.Tm);
  w.total = w.order + round256(4 * cols);
  return w;
}
}  // namespace

extern "C" {

size_t spa2_bwd_rows_workspace_bytes(const spa2_shape* shape) {
  if (check_shape(shape) != SPA2_OK) return 0;
  return rows_ws(make_dims(*shape)).total;
}

int spa2_bwd_rows(const void* q, const void* k, const void* v, const void* o, const void* o_res, const void* d_o,
                  const float* lse, const spa2_shape* shape, const spa2_pattern* pattern, float scale, void* dq, void* dk,
                  void* dv, void* workspace, size_t workspace_bytes, void* stream) {
  const int rc = check_shape(shape);
  if (rc != SPA2_OK) return rc;
  if (!q || !k || !v || !o || !d_o || !lse || !dq || !dk || !dv || !pattern) return SPA2_ERR_NULL;
  if (!pattern->mask || !pattern->row_cnt || !pattern->row_idx) return SPA2_ERR_NULL;
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o) || !aligned16(d_o) || !aligned16(dq) ||
      !aligned16(dk) || !aligned16(dv) || !aligned16(o_res))
    return SPA2_ERR_ALIGN;
  if (!(scale > 0.f) || !isfinite(scale)) return SPA2_ERR_RANGE;
  const Dims m = make_dims(*shape);
  if (m.Tn > SPA2_MAX_TN) return SPA2_ERR_SHAPE;
  const RowsWs w = rows_ws(m);
  if (!workspace || workspace_bytes < w.total) return SPA2_ERR_WORKSPACE;
  if (!aligned16(workspace)) return SPA2_ERR_ALIGN;
  int32_t* col_cnt = (int32_t*)((char*)workspace + w.cnt);
  int32_t* col_idx = (int32_t*)((char*)workspace + w.idx);
  int32_t* col_order = (int32_t*)((char*)workspace + w.order);
  SplitPlan rows = dq_plan(m, workspace, workspace_bytes), cols = dkdv_plan(m, workspace, workspace_bytes);
  cols = columns_in_stretches(cols, m);
  float* delta = (float*)workspace;
  hipStream_t st = (hipStream_t)stream;
  if (m.Tn > SIDE_ORDER_MAX) {            // (262,144 tokens and more: two launches are nothing there)
    if (launch_columns(pattern->mask, m, col_cnt, col_idx, col_order, st) != hipSuccess ||
        launch_bwd_prepare(o, o_res, d_o, m, delta, pattern->row_cnt, rows, col_cnt, cols, st) != hipSuccess)
      return SPA2_ERR_LAUNCH;
  } else if (launch_bwd_prepare_columns(o, o_res, d_o, m, delta, pattern->row_cnt, rows, pattern->mask, col_cnt, col_idx,
                                        st) != hipSuccess) {
    return SPA2_ERR_LAUNCH;
  }
  rows.planned = cols.planned = true;
  const hipError_t e = m.Tn > SIDE_ORDER_MAX
      ? launch_bwd_dq(q, k, v, d_o, lse, delta, m, pattern->row_cnt, pattern->row_idx, pattern->row_order, scale, dq, rows, st)
      : launch_bwd_dq_columns(q, k, v, d_o, lse, delta, m, pattern->row_cnt, pattern->row_idx, pattern->row_order, scale, dq,
                              rows, col_cnt, col_order, cols, st);
  if (e != hipSuccess) return SPA2_ERR_LAUNCH;
  return launch_bwd_dkdv(q, k, v, d_o, lse, delta, m, col_cnt, col_idx, col_order, scale, dk, dv, cols, st) == hipSuccess
             ? SPA2_OK : SPA2_ERR_LAUNCH;
}

}  // extern "C"
