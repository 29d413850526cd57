// Splitting of long rows (columns) of the block pattern over several workgroups.
//
// One workgroup walks one row of the pattern in the forward and dQ kernels (one column in the dK/dV kernel), so a
// launch cannot finish before its longest row has.  On a layer with few rows per workgroup slot the longest rows
// (Top-p-bound rows are ten times the Top-k length) then set the time, and on a small layer there are fewer rows than
// compute units.  This plan cuts every list longer than S entries into equal parts of at most S entries.  The parts
// are workgroups of their own at the front of the same launch; every part leaves an fp32 partial result in a pool slot
// and counts itself in, and the part that arrives last adds up all of them in part order, so results do not depend on
// the order of execution.
//
// The plan is computed on the device from the list lengths (the host never reads the pattern):
//   T = total number of list entries of the launch,
//   S = max(min(max(T / 512, lo), mid), min(T / 2048, 48), T / 8192)   (quotients rounded up),
// with 512 (RESIDENT_WGS) the number of workgroups that run at a time; dK/dV at d = 64 runs 1024, and its divisors are
// twice these.  Small launches are cut until the slots
// are filled, down to lo entries, below which a part is mostly prologue and merge; ordinary ones into quarters of the
// mean work of a slot, but not below mid (parts of 8 instead of 16 cost more than they balance) nor above 48; on the
// largest only lists of more than a sixteenth of a slot's mean work are cut, which the natural launch order would
// otherwise start anywhere up to the end of the launch.
// Measured (us, forward / dQ / dK,dV; before = parts of T / 2048 with part 0 in its row's place and merge kernels):
//   75,600 tokens, 40 heads (T = 1.6 M):  8059 / 11248 / 14926 before, 7600 / 10610 / 14655 now
//   32,760 tokens, 12 heads (T = 91 k):    474 /   615 /   936 before,  445 /   595 /   928 now
//   20,010 tokens, 6 heads, d = 64:         99 /   109 /   184 before,   76 /    93 /   165 now
//   32,760 tokens, 3 heads, every tile:   2267 before, 1663 now
#include "columns.h"
#include "row_delta.h"
#include "spa2_device.h"
#include "spa2_internal.h"
#include "split_plan.h"

namespace spa2 {

namespace {
inline size_t up256(size_t x) { return (x + 255) & ~(size_t)255; }
}

// lo and mid of the rule above.  An entry of a column is twice the work of one of a row.  Measured on 264 rows of 7
// entries (dQ) and 504 columns of 3 to 9: lo = 8 / 4 takes 38 / 61 us, lo = 4 / 2 59 / 61 us, lo = 16 / 8 38 / 64 us;
// on 32 rows of 29 and 64 columns of 14 (d = 64) 28 / 33, 28 / 36 and 34 / 41 us.  The forward kernel cuts that finely
// only where most compute units would have no row at all: its parts round P against their own running maxima, and a
// row of few tiles then shows the other rounding.
static void split_range(SplitKind kind, int64_t units, int& lo, int& mid) {
  if (kind == SPLIT_DKDV) { lo = 4; mid = 12; return; }
  mid = 16;
  lo = kind == SPLIT_DQ || units <= 128 ? 8 : 16;
}

// Pool sizes are powers of two from 8 to SPLIT_POOL_MAX (a multiple of 8 keeps the workgroup -> XCD phase of the
// launch that the parts are put in front of): room for every list to be cut into 16 parts, or as many as it has pairs
// of entries.
static int64_t pool_wanted(int64_t units, int list_max) {
  const int64_t per_unit = list_max / 2 < 1 ? 1 : (list_max / 2 > 16 ? 16 : list_max / 2);
  int64_t pool = 8;
  while (pool < SPLIT_POOL_MAX && pool < per_unit * units) pool *= 2;
  return pool;
}

static size_t tables_bytes(int64_t units, int64_t pool) {
  return 256 + up256((size_t)units * 4) + up256((size_t)pool * 16) + up256((size_t)pool * 4);
}

size_t split_ws_bytes(int64_t units, int list_max, size_t slot_bytes) {
  const int64_t pool = pool_wanted(units, list_max);
  return tables_bytes(units, pool) + (size_t)pool * slot_bytes;
}

size_t split_pool_offset(int64_t units, int list_max) { return tables_bytes(units, pool_wanted(units, list_max)); }

SplitPlan split_layout(void* ws, size_t ws_bytes, int64_t units, int list_max, size_t slot_bytes) {
  SplitPlan p;
  p.header = nullptr; p.unit_slot = nullptr; p.part_table = nullptr; p.arrive = nullptr; p.pool = nullptr;
  p.queue = nullptr;
  p.pool_slots = 0; p.slot_floats = 0; p.fixed_len = 0; p.fixed_parts = 0; p.planned = false;
  p.resident = RESIDENT_WGS; p.stretches = false; p.queue_if_full = false;
  if (!ws) return p;
  // the pool shrinks if the caller gave less than the full workspace
  int64_t pool = pool_wanted(units, list_max);
  while (pool >= 8 && tables_bytes(units, pool) + (size_t)pool * slot_bytes > ws_bytes) pool /= 2;
  if (pool < 8) return p;
  char* c = (char*)ws;
  p.pool_slots = (int)pool;
  p.header = (int32_t*)c;                 c += 256;
  p.unit_slot = (int32_t*)c;              c += up256((size_t)units * 4);
  p.part_table = (int32_t*)c;             c += up256((size_t)pool * 16);
  p.arrive = (int32_t*)c;                 c += up256((size_t)pool * 4);
  p.pool = (float*)c;
  p.slot_floats = (int)(slot_bytes / 4);
  return p;
}

// T <= units * list_max: where that is within 512 lo, S is lo (see above) whatever the lists are.
SplitPlan with_fixed_parts(SplitPlan p, int64_t units, int list_max) {
  int lo, mid;
  split_range(SPLIT_FWD, units, lo, mid);
  const int parts = (list_max + lo - 1) / lo;
  if (p.pool_slots && units * list_max <= (int64_t)RESIDENT_WGS * lo && units * parts <= p.pool_slots) {
    p.fixed_len = lo; p.fixed_parts = parts; p.planned = true;
  }
  return p;
}

PlanArgs plan_args(const int32_t* cnt, int64_t units, int list_max, SplitKind kind, const SplitPlan& p) {
  PlanArgs a;
  a.cnt = cnt; a.units = (int)units; a.list_max = list_max;
  split_range(kind, units, a.lo, a.mid);
  a.pool = kind == SPLIT_DKDV ? p.pool_slots - 1 : p.pool_slots;      // (the last slot is the queue's, whether there is one or not)
  a.queue = p.queue; a.slots_log2 = __builtin_ctz(p.resident); a.eighths = p.stretches;
  a.header = (int32_t*)p.header; a.unit_slot = (int32_t*)p.unit_slot; a.part_table = (int32_t*)p.part_table;
  a.arrive = p.arrive;
  return a;
}

template <int NT>
__global__ __launch_bounds__(NT) void split_plan_kernel(PlanArgs a) {
  __shared__ PlanLds<NT> lds;
  plan_block<NT>(a, lds);
}

hipError_t launch_split_plan(const int32_t* cnt, int64_t units, int list_max, SplitKind kind, const SplitPlan& p,
                             hipStream_t stream) {
  if (p.pool_slots == 0) return hipSuccess;
  const PlanArgs a = plan_args(cnt, units, list_max, kind, p);
  // (one quad of lengths per thread of the small workgroup: 16 units 4.6 -> 3.6 us, 264 units 5.0 -> 3.7 us)
  if (units <= 1024) hipLaunchKernelGGL(split_plan_kernel<256>, dim3(1), dim3(256), 0, stream, a);
  else               hipLaunchKernelGGL(split_plan_kernel<1024>, dim3(1), dim3(1024), 0, stream, a);
  return hipGetLastError();
}

// The pass over O and dO with work of its own workgroups in front of it: the plans of the backward kernels, one workgroup
// each (two launches of 8 to 27 us before), and, where the pattern came without them, the column lists (a launch of 4 to 27
// us before).  Neither costs time of its own wherever the pass takes longer than they do.
struct PrepareArgs { DeltaArgs d; PlanArgs plan[2]; int n_plans; ColumnArgs cols; int n_cols, col_width; };

template <int D>
__global__ __launch_bounds__(256) void bwd_prepare_kernel(PrepareArgs a) {
  __shared__ union { PlanLds<256> plan; int cnt64[4][64], cnt32[8][32], cnt16[16][16]; } lds;
  int w = blockIdx.x;
  if (w < a.n_plans) {
    plan_block<256>(a.plan[w], lds.plan);
    return;
  }
  w -= a.n_plans;
  if (w < a.n_cols) {
    const int bh = w / a.cols.groups, group = w % a.cols.groups;
    if (a.col_width == 64)      columns_block(a.cols, bh, group, lds.cnt64);
    else if (a.col_width == 32) columns_block(a.cols, bh, group, lds.cnt32);
    else                        columns_block(a.cols, bh, group, lds.cnt16);
    return;
  }
  w -= a.n_cols;
  delta_block<D>(a.d, w / a.d.chunks, w % a.d.chunks);
}

static hipError_t launch_prepare(const PrepareArgs& a, const Dims& m, hipStream_t stream) {
  const dim3 grid((unsigned)(a.n_plans + a.n_cols + m.B * m.H * a.d.chunks)), block(256);
  if (m.d == 128) hipLaunchKernelGGL(bwd_prepare_kernel<128>, grid, block, 0, stream, a);
  else            hipLaunchKernelGGL(bwd_prepare_kernel<64>, grid, block, 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_bwd_prepare(const void* o, const void* o_res, const void* d_o, const Dims& m, float* delta,
                              const int32_t* row_cnt, const SplitPlan& row_plan, const int32_t* col_cnt,
                              const SplitPlan& col_plan, hipStream_t stream) {
  PrepareArgs a = {};
  a.d = delta_args(o, o_res, d_o, m, delta);
  if (col_plan.pool_slots) a.plan[a.n_plans++] = plan_args(col_cnt, (int64_t)m.B * m.H * m.Tn, m.Tm, SPLIT_DKDV, col_plan);
  if (row_plan.pool_slots) a.plan[a.n_plans++] = plan_args(row_cnt, (int64_t)m.B * m.H * m.Tm, m.Tn, SPLIT_DQ, row_plan);
  return launch_prepare(a, m, stream);
}

hipError_t launch_bwd_prepare_columns(const void* o, const void* o_res, const void* d_o, const Dims& m, float* delta,
                                      const int32_t* row_cnt, const SplitPlan& row_plan, const uint8_t* mask,
                                      int32_t* col_cnt, int32_t* col_idx, hipStream_t stream) {
  PrepareArgs a = {};
  a.d = delta_args(o, o_res, d_o, m, delta);
  if (row_plan.pool_slots) a.plan[a.n_plans++] = plan_args(row_cnt, (int64_t)m.B * m.H * m.Tm, m.Tn, SPLIT_DQ, row_plan);
  // Columns a workgroup shares.  Long columns (runs of more than 64 query blocks a thread, read in rounds that wait for each
  // other, and a second time) of few heads take longer than D: there fewer columns and more runs.  us, the launch, 64 / 32 / 16:
  // 1 head of 131,072 tokens 30.6 / 18.4 / 13.9, d = 128 37.2 / 25.2 / 21.8, of 262,144 59.1 / 37.4 / 32.0, of 65,536, d = 128
  // 18.8 / 13.0 / 12.7; 2 of 131,072 (64 workgroups) 37.0 / 25.6 / 23.4, 4 48.5 / 39.7 / 42.6, 8 89.0 / 85.9 / 92.4; 4 of 65,536
  // 23.8 / 20.5 / 21.7; 40 of 75,600 (760) 411.9 / 416.1 / 422.2; shorter columns (T_m <= 256): within 0.8 of each other up to 12
  // heads of 32,768, 25.6 / 26.4 / 27.2 there.
  const int64_t wgs = (int64_t)m.B * m.H * ((m.Tn + 63) / 64);
  a.col_width = m.Tm <= 256 || wgs > 128 ? 64 : wgs > 64 ? 32 : 16;
  a.cols = column_args(mask, m, col_cnt, col_idx, a.col_width);
  a.n_cols = m.B * m.H * a.cols.groups;
  return launch_prepare(a, m, stream);
}

}  // namespace spa2
