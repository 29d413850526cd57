// The split plan of one launch, made by one workgroup (see split.hip for what it is): as a launch of its own, or as a
// workgroup of a launch in front of the one that needs it.
#pragma once
#include "spa2_device.h"
#include "spa2_internal.h"

namespace spa2 {

constexpr int SPLIT_CAP = 48;

// What one plan reads and writes.
struct PlanArgs {
  const int32_t* cnt;
  int units, list_max, lo, mid, pool;
  int slots_log2;              // of the workgroups that run at a time
  bool eighths;                // header[2] is read (SplitPlan::stretches)
  int32_t* header; int32_t* unit_slot; int32_t* part_table; int32_t* arrive; int32_t* queue;
};

typedef __attribute__((ext_vector_type(4))) int i32x4;

PlanArgs plan_args(const int32_t* cnt, int64_t units, int list_max, SplitKind kind, const SplitPlan& p);

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
struct PlanLds {
  i32x4 item[SPLIT_POOL_MAX / 2];                    // (unit, first slot, parts, entries per part) of a split unit
  unsigned long long red[NT / 64];
  int wave_slots[NT / 64], wave_items[NT / 64];
  unsigned long long work[8][32];                    // list entries of every eighth of the units, in 32 shares
  uint16_t owner[SPLIT_POOL_MAX];                    // slot -> entry of the list of split units
};
template <int NT>
__device__ __forceinline__ void plan_block(const PlanArgs& a, PlanLds<NT>& lds) {
  auto &red = lds.red;
  auto &wave_slots = lds.wave_slots, &wave_items = lds.wave_items;
  auto &owner = lds.owner;
  auto &item = lds.item;
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
  // The work of the eighths is summed only where it is read, and the shares of the slots are shifts: plan launch, us, without
  // eighths at all / summed always, with divisions / this: 942 units 6.0 / 7.1 / 6.5, 768 6.7 / 8.6 / 8.0, 3072 8.5 / 9.2 / 8.4,
  // 23,640 (nobody reads them) 13.8 / 14.5 / 13.5, 2048 (nobody) 9.0 / 9.7 / 9.2.
  long long T = 0, most = 0;
  if (!a.eighths) {
    unsigned long long mine = 0;
    each_quad([&](int, const i32x4& c) { mine += (unsigned long long)c[0] + c[1] + c[2] + c[3]; });
    T = (long long)block_sum<NT>(mine, red);
  } else {
    // (shares by lane: the 64 atomics of a wave on one counter stand in a row, 942 units 8.0 us)
    for (int x = t; x < 8 * 32; x += NT) lds.work[x / 32][x % 32] = 0;
    __syncthreads();
    const float eighth = 8.f / (float)a.units;
    each_quad([&](int u, const i32x4& c) {
      const int x0 = min((int)((float)u * eighth), 7), x3 = min((int)((float)(u + 3) * eighth), 7);
      if (x0 == x3) atomicAdd(&lds.work[x0][t % 32], (unsigned long long)c[0] + c[1] + c[2] + c[3]);
      else
#pragma unroll
        for (int e = 0; e < 4; ++e) atomicAdd(&lds.work[min((int)((float)(u + e) * eighth), 7)][t % 32], (unsigned long long)c[e]);
    });
    __syncthreads();
    // (every wave adds up all shares: a lane four of one eighth)
    {
      const int x = lane >> 3, k = 4 * (lane & 7);
      T = (long long)(lds.work[x][k] + lds.work[x][k + 1] + lds.work[x][k + 2] + lds.work[x][k + 3]);
#pragma unroll
      for (int off = 1; off < 8; off <<= 1) T += __shfl_xor(T, off, 64);
      most = T;
#pragma unroll
      for (int off = 8; off < 64; off <<= 1) { T += __shfl_xor(T, off, 64); most = max(most, (long long)__shfl_xor(most, off, 64)); }
    }
  }
  auto share = [&](int k) -> long long { return (T + (1ll << k) - 1) >> k; };       // T / 2^k, rounded up
  const long long s_small = min(max(share(a.slots_log2), (long long)a.lo), (long long)a.mid);
  const long long s_large = max(min(share(a.slots_log2 + 2), (long long)SPLIT_CAP), share(a.slots_log2 + 4));
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
  if (t == 0) {
    a.header[0] = n; a.header[1] = S;
    a.header[2] = 8 * most <= T + T / 16 ? 1 : 0;      // (1 where nobody asks)
    a.header[3] = 16 * T >= 15ll * a.units * a.list_max ? 1 : 0;
  }
  if (a.queue && t < 8) a.queue[t * QUEUE_STRIDE] = 1 << (a.slots_log2 - 3);      // (the first ones go by workgroup number)
}

}  // namespace spa2
