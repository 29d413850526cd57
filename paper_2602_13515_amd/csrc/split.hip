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
// with 512 (RESIDENT_WGS) the number of workgroups that run at a time.  Small launches are cut until the slots
// are filled, down to lo entries, below which a part is mostly prologue and merge; ordinary ones into quarters of the
// mean work of a slot, but not below mid (parts of 8 instead of 16 cost more than they balance) nor above 48; on the
// largest only lists of more than a sixteenth of a slot's mean work are cut, which the natural launch order would
// otherwise start anywhere up to the end of the launch.
// Measured (us, forward / dQ / dK,dV; before = parts of T / 2048 with part 0 in its row's place and merge kernels):
//   75,600 tokens, 40 heads (T = 1.6 M):  8059 / 11248 / 14926 before, 7600 / 10610 / 14655 now
//   32,760 tokens, 12 heads (T = 91 k):    474 /   615 /   936 before,  445 /   595 /   928 now
//   20,010 tokens, 6 heads, d = 64:         99 /   109 /   184 before,   76 /    93 /   165 now
//   32,760 tokens, 3 heads, every tile:   2267 before, 1663 now
#include "row_delta.h"
#include "spa2_device.h"
#include "spa2_internal.h"

namespace spa2 {

namespace {
inline size_t up256(size_t x) { return (x + 255) & ~(size_t)255; }
}

constexpr int SPLIT_CAP = 48;
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

// What one plan reads and writes.
struct PlanArgs {
  const int32_t* cnt;
  int units, list_max, lo, mid, pool;
  int32_t* header; int32_t* unit_slot; int32_t* part_table; int32_t* arrive; int32_t* queue;
};

static PlanArgs plan_args(const int32_t* cnt, int64_t units, int list_max, SplitKind kind, const SplitPlan& p) {
  PlanArgs a;
  a.cnt = cnt; a.units = (int)units; a.list_max = list_max;
  split_range(kind, units, a.lo, a.mid);
  a.pool = p.queue ? p.pool_slots - 1 : p.pool_slots;
  a.queue = p.queue;
  a.header = (int32_t*)p.header; a.unit_slot = (int32_t*)p.unit_slot; a.part_table = (int32_t*)p.part_table;
  a.arrive = p.arrive;
  return a;
}

typedef __attribute__((ext_vector_type(4))) int i32x4;

// Sum over the NT threads of a workgroup (red: one entry per wave).
template <int NT>
__device__ __forceinline__ unsigned long long block_sum(unsigned long long x, unsigned long long* red) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
  __syncthreads();                                   // (the previous sum has been read)
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
  __syncthreads();
  unsigned long long t = 0;
#pragma unroll
  for (int i = 0; i < NT / 64; ++i) t += red[i];
  return t;
}

// Number of parts of at most S entries that a list of c entries is cut into (0: it is not cut).  inv_s = 1 / S; the
// rounded quotient is off by one at most (c < 2^25 entries, S of at least 4 for lists that long) and put right.
__device__ __forceinline__ int parts_of(int c, int S, float inv_s) {
  if (c <= S) return 0;
  int q = (int)((float)c * inv_s);
  q += q * S < c ? 1 : 0;
  q += q * S < c ? 1 : 0;
  return q - ((q - 1) * S >= c ? 1 : 0);
}

// One workgroup of NT threads makes one plan: sum of the lengths (fixes S), number of parts at S (S grows until they
// fit the pool), then every split unit gets its slots by a scan over the threads.
// Bound: latency, of three passes over the lengths (each thread's first four stay in registers) and of fetching the
// code, which every launch runs once: it is kept short (four sizes S a round, unrolled, took 6.4 us instead of 3.6 on
// 16 units).  Slots come from a scan: LDS counters, which every split unit added to, took 20 us instead of 13 for the
// columns of a 20,010-token layer (256 threads).
template <int NT>
__device__ __forceinline__ void plan_block(const PlanArgs& a) {
  __shared__ unsigned long long red[NT / 64];
  __shared__ int wave_slots[NT / 64], wave_items[NT / 64];
  __shared__ uint16_t owner[SPLIT_POOL_MAX];         // slot -> entry of the list of split units
  __shared__ i32x4 item[SPLIT_POOL_MAX / 2];         // (unit, first slot, parts, entries per part) of a split unit
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const bool vec_ok = ((uintptr_t)a.cnt & 15) == 0;
  auto load4 = [&](int u) -> i32x4 {                 // lengths of units u .. u+3 (0 past the end), clamped
    i32x4 c = {0, 0, 0, 0};
    if (vec_ok && u + 4 <= a.units) c = *(const i32x4*)(a.cnt + u);
    else {
#pragma unroll
      for (int x = 0; x < 4; ++x) if (u + x < a.units) c[x] = a.cnt[u + x];
    }
#pragma unroll
    for (int x = 0; x < 4; ++x) c[x] = min(max(c[x], 0), a.list_max);
    return c;
  };
  const i32x4 held = load4(4 * t);
  auto each_quad = [&](auto&& f) {                   // f(first unit, lengths) for every quad of this thread, in order
    i32x4 c = held, next = {0, 0, 0, 0};
#pragma unroll 1
    for (int u = 4 * t; u < a.units; u += 4 * NT, c = next) {
      if (u + 4 * NT < a.units) next = load4(u + 4 * NT);
      f(u, c);
    }
  };
  unsigned long long mine = 0;
  each_quad([&](int, const i32x4& c) { mine += (unsigned long long)c[0] + c[1] + c[2] + c[3]; });
  const long long T = (long long)block_sum<NT>(mine, red);
  const long long s_small = min(max((T + RESIDENT_WGS - 1) / RESIDENT_WGS, (long long)a.lo), (long long)a.mid);
  const long long s_large = max(min((T + 2047) / 2048, (long long)SPLIT_CAP), (T + 8191) / 8192);
  int S = (int)max(min(max(s_small, s_large), (long long)a.list_max), 1ll);
  float inv_s;
  int n_slots, n_items;                              // of this thread's units
#pragma unroll 1
  for (;;) {
    inv_s = 1.f / (float)S;
    n_slots = 0; n_items = 0;
    each_quad([&](int, const i32x4& c) {
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        n_slots = min(n_slots + parts_of(c[x], S, inv_s), 1 << 20);         // (more than any pool: no overflow)
        n_items += c[x] > S ? 1 : 0;
      }
    });
    const int total = (int)block_sum<NT>((unsigned long long)n_slots, red);
    if (total <= a.pool) break;
    // half of what would bring lists much longer than S down to the pool, a quarter at least (ends: no list is longer
    // than list_max)
    S += max(S / 4 + 1, (int)min(0.5f * (float)S * (float)(total - a.pool) / (float)a.pool, (float)S));
  }
  // slots and places in the list of split units: exclusive scan over the threads
  int at_slot = n_slots, at_item = n_items;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int ys = __shfl_up(at_slot, off, 64), yi = __shfl_up(at_item, off, 64);
    if (lane >= off) { at_slot += ys; at_item += yi; }
  }
  if (lane == 63) { wave_slots[w] = at_slot; wave_items[w] = at_item; }
  at_slot -= n_slots; at_item -= n_items;
  __syncthreads();
  int n = 0;
#pragma unroll
  for (int x = 0; x < NT / 64; ++x) {
    if (x < w) { at_slot += wave_slots[x]; at_item += wave_items[x]; }
    n += wave_slots[x];
  }
  each_quad([&](int u, const i32x4& c) {
    i32x4 slot;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      slot[x] = -1;
      if (c[x] > S) {
        const int parts = parts_of(c[x], S, inv_s);
        slot[x] = at_slot;
        item[at_item] = i32x4{u + x, at_slot, parts, (c[x] + parts - 1) / parts};
        for (int p = 0; p < parts; ++p) owner[at_slot + p] = (uint16_t)at_item;
        at_slot += parts; ++at_item;
      }
    }
    if (u + 4 <= a.units) *(i32x4*)(a.unit_slot + u) = slot;
    else {
#pragma unroll
      for (int x = 0; x < 4; ++x) if (u + x < a.units) a.unit_slot[u + x] = slot[x];
    }
  });
  __syncthreads();
  for (int g = t; g < n; g += NT) {
    const i32x4 it = item[owner[g]];
    *(i32x4*)(a.part_table + 4 * g) = i32x4{it[0], g - it[1], it[2], it[3]};
    a.arrive[g] = 0;
  }
  if (t == 0) { a.header[0] = n; a.header[1] = S; }
  if (a.queue && t < 8) a.queue[t * QUEUE_STRIDE] = RESIDENT_WGS / 8;      // (the first ones go by workgroup number)
}

template <int NT>
__global__ __launch_bounds__(NT) void split_plan_kernel(PlanArgs a) { plan_block<NT>(a); }

hipError_t launch_split_plan(const int32_t* cnt, int64_t units, int list_max, SplitKind kind, const SplitPlan& p,
                             hipStream_t stream) {
  if (p.pool_slots == 0) return hipSuccess;
  const PlanArgs a = plan_args(cnt, units, list_max, kind, p);
  // (one quad of lengths per thread of the small workgroup: 16 units 4.6 -> 3.6 us, 264 units 5.0 -> 3.7 us)
  if (units <= 1024) hipLaunchKernelGGL(split_plan_kernel<256>, dim3(1), dim3(256), 0, stream, a);
  else               hipLaunchKernelGGL(split_plan_kernel<1024>, dim3(1), dim3(1024), 0, stream, a);
  return hipGetLastError();
}

// The pass over O and dO with the two plans of the backward kernels in front of it (workgroups 0 .. n_plans-1): the
// plans, one workgroup each, then cost no time of their own (two launches of 8 to 27 us before) wherever the pass
// takes longer than they do.
struct PrepareArgs { DeltaArgs d; PlanArgs plan[2]; int n_plans; };

template <int D>
__global__ __launch_bounds__(256) void bwd_prepare_kernel(PrepareArgs a) {
  if ((int)blockIdx.x < a.n_plans) {
    plan_block<256>(a.plan[blockIdx.x]);
    return;
  }
  const int w = blockIdx.x - a.n_plans;
  delta_block<D>(a.d, w / a.d.chunks, w % a.d.chunks);
}

hipError_t launch_bwd_prepare(const void* o, const void* o_res, const void* d_o, const Dims& m, float* delta,
                              const int32_t* row_cnt, const SplitPlan& row_plan, const int32_t* col_cnt,
                              const SplitPlan& col_plan, hipStream_t stream) {
  PrepareArgs a;
  a.d = delta_args(o, o_res, d_o, m, delta);
  a.n_plans = 0;
  if (col_plan.pool_slots) a.plan[a.n_plans++] = plan_args(col_cnt, (int64_t)m.B * m.H * m.Tn, m.Tm, SPLIT_DKDV, col_plan);
  if (row_plan.pool_slots) a.plan[a.n_plans++] = plan_args(row_cnt, (int64_t)m.B * m.H * m.Tm, m.Tn, SPLIT_DQ, row_plan);
  for (int x = a.n_plans; x < 2; ++x) a.plan[x] = PlanArgs{};
  const dim3 grid((unsigned)(a.n_plans + m.B * m.H * a.d.chunks)), block(256);
  if (m.d == 128) hipLaunchKernelGGL(bwd_prepare_kernel<128>, grid, block, 0, stream, a);
  else            hipLaunchKernelGGL(bwd_prepare_kernel<64>, grid, block, 0, stream, a);
  return hipGetLastError();
}

}  // namespace spa2
