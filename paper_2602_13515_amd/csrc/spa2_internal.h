// Host-side declarations shared by the spa2 translation units (not part of the ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "spa2.h"

namespace spa2 {

struct Dims {
  int B, H, N, d, Tm, Tn;
  int64_t sb, sh, sn;
};

inline Dims make_dims(const spa2_shape& s) {
  Dims m;
  m.B = s.B; m.H = s.H; m.N = s.N; m.d = s.d;
  m.Tm = (s.N + SPA2_BQ - 1) / SPA2_BQ;
  m.Tn = (s.N + SPA2_BKV - 1) / SPA2_BKV;
  m.sb = s.sb; m.sh = s.sh; m.sn = s.sn;
  return m;
}

// Splitting of long rows / columns over several workgroups (split.hip).  All pointers lie in the caller's
// workspace; pool_slots == 0 means "no splitting" and every other member is then null.
constexpr int SPLIT_POOL_MAX = 2048;         // partial-result slots of one launch at most
constexpr int QUEUE_STRIDE = 64;             // ints between the counters of two XCDs (atomics on one line stand in a row)
// Workgroups that run at a time, two per compute unit (fwd_kernel<64>, whose registers and LDS would let three, is cut and
// ordered for two as well): those of a queue launch, and what the split plan cuts for.
constexpr int RESIDENT_WGS = 512;
inline int dkdv_resident(const Dims& m) { return m.d == 128 ? RESIDENT_WGS : 2 * RESIDENT_WGS; }     // (of the dK/dV kernel)
constexpr int SIDE_ORDER_MAX = 4096;         // columns that a side workgroup orders: their keys have to fit the LDS of tiles
struct SplitPlan {
  const int32_t* header;       // [0] number of parts, [1] S = list entries per part at most (for inspection), [2] see stretches,
                               // [3] see queue_if_full
  const int32_t* unit_slot;    // [units] first pool slot of a split unit (its part p uses slot + p), -1 if not split
  const int32_t* part_table;   // [pool_slots][4] (unit, part, parts of the unit, list entries per part) of pool slot g
  int32_t* arrive;             // [pool_slots] parts of the unit that have left their result, at its first slot
  float* pool;                 // [pool_slots][slot_floats] fp32 partial results
  int32_t* queue;              // counters of a queue launch (work_queue.h), QUEUE_STRIDE apart, in the last slot's place; or
                               // null: direct launch
  bool queue_if_full;          // header[3] says whether the launch, as large as a direct one, draws from the queue (with_queue)
  int pool_slots;
  int slot_floats;
  int fixed_len;               // > 0: no plan, every list is cut into parts of at most fixed_len entries (with_fixed_parts);
  int fixed_parts;             //   part p of unit u has slot u * fixed_parts + p
  int resident;                // workgroups of the launch that run at a time
  bool stretches;              // header[2] says whether an XCD takes an eighth of all rows or of every head (with_stretches)
  bool planned;                // the tables have been written already (launch_bwd_prepare): no plan launch of its own
};
// Which rows an XCD takes, where heads are short: an eighth of all rows, one head after the other, so that the workgroups that
// run on an XCD at a time are of one head or a few, whose keys and values its 4 MB of L2 then serve.  (With an eighth of every
// head on every XCD the 64 workgroups of an XCD were of 16 heads where a head has 32 rows.)  Where heads are of unlike density,
// so that an eighth has a sixteenth more list entries than the mean, an eighth of every head is what evens out: the plan says
// which (header[2]).  From 512 rows an eighth of a head fills an XCD as well.  Measured, us, an eighth of every head / of all
// (forward, dQ): 24 heads of 4000 tokens 45.2 / 39.0, 44.2 / 42.1; 16 heads of 8192 75.4 / 70.7, 82.7 / 81.0; 32 heads of 8192, d = 64
// 202.7 / 194.3, 225.9 / 224.1; 24 heads of 32,760 846 / 841, 1025 / 1014, d = 64 487 / 478, 610 / 602; 384 rows: 12 heads of 49,152
// 945 / 947, 1140 / 1140, d = 64 526 / 517, 645 / 640; 511 rows: 6 of 65,408 810 / 808, 988 / 1002, d = 64 468 / 484, 585 / 586; 591:
// 12 of 75,600 1996 / 2045, 2641 / 2637, d = 64 1237 / 1245, 1463 / 1485; 1024: 4 of 131,072 2055 / 2127, 2686 / 2634, d = 64 1222 /
// 1224, 1418 / 1453.
inline SplitPlan with_stretches(SplitPlan p, const Dims& m) {
  p.stretches = p.pool_slots && m.Tm < 512;
  return p;
}
// Whether a launch draws its units from a queue (work_queue.h): where every workgroup gets more than four.  dK/dV, direct /
// queue, us, d = 128: 750 columns 51.6 / 59.3 and 66.0 / 72.8, 1500 105.0 / 103.6 and 153.4 / 155.1, 3000 289 / 280.  d = 64, a
// twentieth of the tiles, half the rows long, nine tenths of the tiles: 1536 columns 47 / 62, 127 / 130, 407 / 400; 3584 100 / 102,
// 252 / 257, 850 / 809; 4096 110 / 115, 286 / 292, 907 / 938; 5120 127 / 136, 354 / 355, 1134 / 1191; 8192 197 / 204, 562 / 562, 1814 /
// 1862; 12,288 288 / 296, 863 / 864, 2694 / 2731; and in heads of 32,768 tokens 5120 378 / 393, 1519 / 1497, 4628 / 4767; 8192 543 /
// 563, 2652 / 2447, 7442 / 7313; 12,288 791 / 816, 3922 / 3571, 10,932 / 10,859.  (Beyond the line the queue evens out long columns, up
// to a tenth, and costs short ones a twentieth.)
// At d = 64 (1024 at a time) also where the columns are long and of full length, or nearly (the plan says so: header[3]), and the
// last round of a direct launch would be up to three quarters full: all end at a time there, and the last round's workgroups go
// four to the compute units that are free first.  Every tile, us, direct / queue [one wave a SIMD, in 3 rounds of 512 instead of
// 1.5]: 12 heads of 8192 458 / 416 [421], 11 447 / 400 [406], 18 633 / 591 [673], 24 of 4000 236 / 214 [223], 3 of 32,768 1793 / 1620
// [1564], 48 of 2048 126 / 116 [133]; 14 of 8192 (three quarters full) 500 / 505, 16 (full) 522 / 522, 32 1038 / 1075; 96 heads of 1024
// (8 query blocks) 70 / 66, 72 55 / 58, 600 of 128 17 / 23.  Nine tenths of the tiles: 24 of 4000 210 / 217, 12 of 8192 404 / 382; half
// 123 / 125, 227 / 224; a tenth or less 33 / 47, 47 / 62.
inline SplitPlan with_queue(SplitPlan p, int64_t units, int list_max, int resident) {
  p.resident = resident;
  const bool always = units > 4 * resident;
  const int64_t last = units % resident;
  p.queue_if_full = !always && resident > RESIDENT_WGS && list_max >= 16 && units > resident && last && 4 * last <= 3 * resident;
  if (p.pool_slots && (always || p.queue_if_full)) p.queue = (int32_t*)(p.pool + (size_t)(p.pool_slots - 1) * p.slot_floats);
  return p;
}
// Columns in stretches, where spa2_bwd_rows lists them for it: heads as above, and stretches whose columns a workgroup can rank.
// (Eighths of unlike work: a direct launch takes the stretches in turn, a queue evens out by itself.)  Measured, us, backward
// pass, an eighth of every head / of all: 4 samples of 1281 tokens, 6 heads 73.8 / 68.7; 24 heads of 4000 145.2 / 120.2; 6 heads
// of 9000 165.3 / 154.7; 16 heads of 8192 269 / 246; 40 heads of 3000, d = 64 132.5 / 115.0; 20,010 tokens, 6 heads, d = 64 183.6 /
// 176.4; 24 heads of 32,760 2805 / 2728, half the rows long 12470 / 12170.  The line at 512 rows is that of the length in the list's
// keys; dK/dV would gain beyond it too: 12 heads of 65,408 (511 rows) 3137 / 2975, 12 of 75,600 (591) 4038 / 3882, 4 of 131,072 (1024),
// d = 64 2086 / 1906.
inline SplitPlan columns_in_stretches(SplitPlan p, const Dims& m) {
  p.stretches = p.pool_slots && m.Tm < 512 && (int64_t)m.B * m.H * m.Tn <= 8 * SIDE_ORDER_MAX;
  return p;
}
size_t split_ws_bytes(int64_t units, int list_max, size_t slot_bytes);
size_t split_pool_offset(int64_t units, int list_max);       // where the slots of a full workspace begin
SplitPlan split_layout(void* ws, size_t ws_bytes, int64_t units, int list_max, size_t slot_bytes);
// Plan of the launch of kernel `kind`, which walks `units` lists of at most list_max entries.
enum SplitKind { SPLIT_FWD, SPLIT_DQ, SPLIT_DKDV };
hipError_t launch_split_plan(const int32_t* cnt, int64_t units, int list_max, SplitKind kind, const SplitPlan& p,
                             hipStream_t stream);
// The forward kernel's parts without a plan, where the sizes alone say that the plan would cut into pieces of its least length (and the
// slots suffice): p with fixed_len set.  The caller zeroes p.arrive before the launch.
SplitPlan with_fixed_parts(SplitPlan p, int64_t units, int list_max);
// D = rowsum(dO * O) and the plans of the two backward kernels in one launch (split.hip).
hipError_t launch_bwd_prepare(const void* o, const void* o_res, const void* d_o, const Dims& m, float* delta,
                              const int32_t* row_cnt, const SplitPlan& row_plan, const int32_t* col_cnt,
                              const SplitPlan& col_plan, hipStream_t stream);

// D, the plan of the dQ kernel and the pattern's column lists in one launch; and the dQ launch that makes the plan and the
// launch order (col_order, or null) of the dK/dV kernel on its way (bwd.hip).
hipError_t launch_bwd_prepare_columns(const void* o, const void* o_res, const void* d_o, const Dims& m, float* delta,
                                      const int32_t* row_cnt, const SplitPlan& row_plan, const uint8_t* mask,
                                      int32_t* col_cnt, int32_t* col_idx, hipStream_t stream);
// (heads of up to SIDE_ORDER_MAX columns)
hipError_t launch_bwd_dq_columns(const void* q, const void* k, const void* v, const void* d_o, const float* lse,
                                 const float* delta, const Dims& m, const int32_t* row_cnt, const int32_t* row_idx,
                                 const int32_t* row_order, float scale, void* dq, const SplitPlan& plan,
                                 const int32_t* col_cnt, int32_t* col_order, const SplitPlan& col_plan, hipStream_t stream);

// Each launcher enqueues its kernels on `stream` and returns hipGetLastError().
hipError_t launch_pool(const void* q, const void* k, const Dims& m, float* qbar, float* kbar, hipStream_t stream);
// the same, and zeroes `zeros` integers at `zero` (at most one per thread of the launch)
hipError_t launch_pool_zero(const void* q, const void* k, const Dims& m, float* qbar, float* kbar, int32_t* zero, int zeros,
                            hipStream_t stream);
hipError_t launch_select(const float* qbar, const float* kbar, const Dims& m, int topk_blocks, float top_p,
                         float scale, uint8_t* mask, int32_t* row_cnt, int32_t* row_idx, float* pbar_out,
                         hipStream_t stream);
hipError_t launch_columns(const uint8_t* mask, const Dims& m, int32_t* col_cnt, int32_t* col_idx,
                          int32_t* col_order, hipStream_t stream);
hipError_t launch_pattern_full(const Dims& m, uint8_t* mask, int32_t* row_cnt, int32_t* row_idx,
                               int32_t* col_cnt, int32_t* col_idx, int32_t* col_order, hipStream_t stream);
size_t fwd_slot_bytes(const Dims& m);
hipError_t launch_fwd(const void* q, const void* k, const void* v, const Dims& m, const int32_t* row_cnt,
                      const int32_t* row_idx, const int32_t* row_order, float scale, void* o, void* o_res,
                      float* lse, const SplitPlan& plan, hipStream_t stream);
hipError_t launch_bwd_delta(const void* o, const void* o_res, const void* d_o, const Dims& m, float* delta,
                            hipStream_t stream);
size_t dq_slot_bytes(const Dims& m);
size_t dkdv_slot_bytes(const Dims& m);
hipError_t launch_bwd_dq(const void* q, const void* k, const void* v, const void* d_o, const float* lse,
                         const float* delta, const Dims& m, const int32_t* row_cnt, const int32_t* row_idx,
                         const int32_t* row_order, float scale, void* dq, const SplitPlan& plan, hipStream_t stream);
hipError_t launch_bwd_dkdv(const void* q, const void* k, const void* v, const void* d_o, const float* lse,
                           const float* delta, const Dims& m, const int32_t* col_cnt, const int32_t* col_idx,
                           const int32_t* col_order, float scale, void* dk, void* dv, const SplitPlan& plan,
                           hipStream_t stream);

size_t error_ws_bytes(const Dims& m);
hipError_t launch_error_terms(const void* o_sparse, const void* o_dense, const float* lse_sparse,
                              const float* lse_dense, const Dims& m, double* out, void* ws, hipStream_t stream);

size_t vd_ws_bytes();
hipError_t launch_vd_loss(const void* u_sparse, const void* u_full, int64_t n, bool bf16, double weight, double* loss,
                          void* ws, hipStream_t stream);
hipError_t launch_vd_grad(const void* u_sparse, const void* u_full, int64_t n, bool bf16, double weight,
                          const double* upstream, void* grad, hipStream_t stream);
hipError_t launch_vd_loss_grad(const float* u_sparse, const float* u_full, int64_t n, double weight, double* loss, float* grad,
                               void* ws, hipStream_t stream);
hipError_t launch_vd_rescale(float* grad, int64_t n, double weight, const double* upstream, hipStream_t stream);

}  // namespace spa2
