// Argument checks and workspace layout that several entry points share (host side).
#pragma once
#include <math.h>

#include "spa2_internal.h"

namespace spa2 {

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline size_t round256(size_t x) { return (x + 255) & ~(size_t)255; }

inline int check_shape(const spa2_shape* s) {
  if (!s) return SPA2_ERR_NULL;
  if (s->B <= 0 || s->H <= 0 || s->N <= 0 || s->d <= 0) return SPA2_ERR_SHAPE;
  if (s->bq != SPA2_BQ || s->bkv != SPA2_BKV) return SPA2_ERR_UNSUPPORTED;
  if (s->d != 64 && s->d != 128) return SPA2_ERR_UNSUPPORTED;
  if (s->sb <= 0 || s->sh <= 0 || s->sn < s->d) return SPA2_ERR_SHAPE;
  if ((s->sb % 8) || (s->sh % 8) || (s->sn % 8)) return SPA2_ERR_ALIGN;
  // the kernels address a tile as a 64-bit base plus a 32-bit byte offset of up to 128 token rows
  if (s->sn > SPA2_MAX_TOKEN_STRIDE) return SPA2_ERR_SHAPE;
  if ((int64_t)s->B * s->H > (int64_t)1 << 24) return SPA2_ERR_SHAPE;
  // one-dimensional grids of up to B*H*(T_m + T_n + 16) workgroups, 32-bit workgroup arithmetic in the kernels
  const int64_t tm = ((int64_t)s->N + SPA2_BQ - 1) / SPA2_BQ, tn = ((int64_t)s->N + SPA2_BKV - 1) / SPA2_BKV;
  if ((int64_t)s->B * s->H * (tm + tn + 16) > (int64_t)0x7fffffff) return SPA2_ERR_SHAPE;
  return SPA2_OK;
}

struct MaskWs { size_t qbar, kbar, total; };
inline MaskWs mask_ws(const Dims& m) {
  MaskWs w;
  const size_t bh = (size_t)m.B * m.H;
  w.qbar = 0;
  w.kbar = round256(bh * m.Tm * m.d * sizeof(float));
  w.total = w.kbar + round256(bh * m.Tn * m.d * sizeof(float));
  return w;
}

// Backward workspace: D (fp32, one value per token row), then the split plans and partial-result pools of the dQ
// and the dK/dV kernel.  Only D is mandatory: with less than the full size the kernels walk every list whole.
struct BwdWs { size_t d_bytes, dq_off, dq_bytes, dkdv_off, dkdv_bytes, total; };
inline BwdWs bwd_ws(const Dims& m) {
  BwdWs w;
  w.d_bytes = round256((size_t)m.B * m.H * m.N * sizeof(float));
  w.dq_off = w.d_bytes;
  w.dq_bytes = round256(split_ws_bytes((int64_t)m.B * m.H * m.Tm, m.Tn, dq_slot_bytes(m)));
  w.dkdv_off = w.dq_off + w.dq_bytes;
  w.dkdv_bytes = round256(split_ws_bytes((int64_t)m.B * m.H * m.Tn, m.Tm, dkdv_slot_bytes(m)));
  w.total = w.dkdv_off + w.dkdv_bytes;
  return w;
}
inline size_t bwd_ws_min_bytes(const Dims& m) { return bwd_ws(m).d_bytes; }

// the part of a workspace section that the caller's buffer really covers
inline SplitPlan section_plan(void* ws, size_t ws_bytes, size_t off, size_t bytes, int64_t units, int list_max,
                              size_t slot_bytes) {
  if (!ws || ws_bytes <= off) return split_layout(nullptr, 0, units, list_max, slot_bytes);
  const size_t have = ws_bytes - off < bytes ? ws_bytes - off : bytes;
  return split_layout((char*)ws + off, have, units, list_max, slot_bytes);
}
inline SplitPlan dq_plan(const Dims& m, void* ws, size_t ws_bytes) {
  const BwdWs w = bwd_ws(m);
  return with_stretches(section_plan(ws, ws_bytes, w.dq_off, w.dq_bytes, (int64_t)m.B * m.H * m.Tm, m.Tn, dq_slot_bytes(m)), m);
}
inline SplitPlan dkdv_plan(const Dims& m, void* ws, size_t ws_bytes) {
  const BwdWs w = bwd_ws(m);
  const int64_t units = (int64_t)m.B * m.H * m.Tn;
  return with_queue(section_plan(ws, ws_bytes, w.dkdv_off, w.dkdv_bytes, units, m.Tm, dkdv_slot_bytes(m)), units, m.Tm, dkdv_resident(m));
}

// what spa2_mask asks of everything but its workspace
inline int check_mask(const void* q, const void* k, const spa2_shape* shape, int32_t topk_blocks, float top_p, float scale,
                      const spa2_pattern* out) {
  const int rc = check_shape(shape);
  if (rc != SPA2_OK) return rc;
  if (!q || !k || !out || !out->mask || !out->row_cnt || !out->row_idx) return SPA2_ERR_NULL;
  if ((out->col_cnt == nullptr) != (out->col_idx == nullptr)) return SPA2_ERR_NULL;
  if (!aligned16(q) || !aligned16(k)) return SPA2_ERR_ALIGN;
  const Dims m = make_dims(*shape);
  if (m.Tn > SPA2_MAX_TN) return SPA2_ERR_SHAPE;
  if (topk_blocks < 0 || topk_blocks > m.Tn) return SPA2_ERR_RANGE;
  if (!(top_p >= 0.f) || !(top_p <= 1.f)) return SPA2_ERR_RANGE;
  if (topk_blocks == 0 && top_p == 0.f) return SPA2_ERR_RANGE;
  if (!(scale > 0.f) || !isfinite(scale)) return SPA2_ERR_RANGE;
  return SPA2_OK;
}

// what spa2_fwd asks of everything but its workspace
inline int check_fwd(const void* q, const void* k, const void* v, const spa2_shape* shape, const spa2_pattern* pattern,
                     float scale, const void* o, const void* o_res, const float* lse) {
  const int rc = check_shape(shape);
  if (rc != SPA2_OK) return rc;
  if (!q || !k || !v || !o || !lse || !pattern || !pattern->row_cnt || !pattern->row_idx) return SPA2_ERR_NULL;
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o) || !aligned16(o_res)) return SPA2_ERR_ALIGN;
  if (!(scale > 0.f) || !isfinite(scale)) return SPA2_ERR_RANGE;
  return SPA2_OK;
}

}  // namespace spa2
