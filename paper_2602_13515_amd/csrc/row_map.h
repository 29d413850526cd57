// Which row a workgroup of the forward and dQ kernels takes.
#pragma once
#include "spa2_device.h"
#include "spa2_internal.h"

namespace spa2 {

// The row that workgroup wg behind the parts takes, and how many there are of these (room for either order).
inline int launched_rows(int heads, int rows_per_head, int chunk) {
  const int s = stretch_wgs(heads * rows_per_head), e = xcd_map_wgs(heads, rows_per_head, chunk, SHORT_ROWS);
  return s > e ? s : e;
}
__device__ __forceinline__ HeadBlock launched_row(const SplitPlan& sp, int wg, int heads, int rows_per_head, int chunk) {
  if (sp.stretches && scalar_ld(sp.header + 2) != 0) return stretch_row(wg, heads, rows_per_head);
  HeadBlock r = xcd_map_rows(wg, rows_per_head, chunk);
  r.valid = r.valid && wg < xcd_map_wgs(heads, rows_per_head, chunk, SHORT_ROWS);
  return r;
}
}  // namespace spa2
