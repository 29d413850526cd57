// Which column (or part of one) a workgroup of the dK/dV kernel works on, and which one next.
//
// A launch has one item per column that is not split, and one per part of a split column.  Items are dealt to the eight
// XCDs: parts round-robin, columns by xcd_map or in stretches (columns_in_stretches), in both kinds of launch.
//   * Direct launch: one workgroup per item, the parts first.  For launches that fit the chip at once, and where the
//     caller gave no workspace.
//   * Queue launch (sp.queue, see with_queue): as many workgroups as the compute units hold stay for the whole launch and take items of
//     their XCD, in the same order, from a counter in the workspace that the plan has set; when their XCD has none left
//     they take items of the XCD that has most.
// Why the queue: the dispatcher deals the workgroups of an XCD to its shader engines in turn and in order, and an engine
// that is full holds back the ones behind it: a slot stood empty for 14 us between two workgroups, 9 % of the launch.  The
// next item is drawn before the sums of the present one are exchanged and stored, so that the atomic's way to memory and
// back costs nothing.  Measured, us, direct / queue: 75,600 tokens, 40 heads 13528 / 12936; 32,760 tokens, 12 heads 873 /
// 851; 32,768 tokens, 24 heads, half the rows long 7540 / 7153 (d = 64: see with_queue).  The forward and
// dQ kernels gain less (their launches are bound by power, an empty slot is clock for the others: 1.6 % for dQ, 0.3 % for
// forward on the first of these) and lose on shorter launches (dQ on 20,010 tokens, 6 heads, d = 64 75 / 81): they are launched directly.
// Numbers that stand for no column are drawn as well, an atomic and two barriers each, so the queue has xcd_map's few: with
// chunks of a head on every XCD, heads of less than eight columns left XCDs of nothing but such numbers.  Stage call, us,
// chunks / xcd_map / direct, d = 128: 2,300 heads of one column 113 / 83 / 82; 1,000 heads of 9 columns 324 / 301 / 307.
#pragma once
#include "spa2_device.h"
#include "spa2_internal.h"

namespace spa2 {

// The lane's number, counted anew where it is asked for: a kernel that walks several items keeps no vector register for it
// (nor for what follows from it) across them.
__device__ __forceinline__ int fresh_lane() {
  int ones = -1;
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+s"(ones));
#endif
  return (int)__builtin_amdgcn_mbcnt_hi(ones, __builtin_amdgcn_mbcnt_lo(ones, 0));
}

struct WorkItem {
  int bh, blk;                     // head and key block
  int part, parts, part_len;       // parts == 0: the whole list
  int slot;                        // pool slot of this part
};

// The walk of one workgroup over its items (uniform; every thread makes every call):
//   Walk w(word, sp); while (w.take(...)) { ... w.draw(sp) near the end ...; w.advance(sp) }
// word: LDS of the caller's that is free between the barriers that advance() contains.
struct Walk {
  int xcd, q, drawn;
  int wave;                        // number of the calling wave (scalar)
  bool out;                        // a draw is on its way
  bool queued;
  int* word;

  __device__ __forceinline__ Walk(int* lds_word, const SplitPlan& sp)
      : xcd(blockIdx.x & 7), q(blockIdx.x >> 3), drawn(0), wave(__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)),
        out(false), queued(sp.queue && (!sp.queue_if_full || scalar_ld(sp.header + 3) != 0)), word(lds_word) {}

  // a workgroup beyond those that stay, in a launch that was made for both ways (queue_if_full)
  __device__ __forceinline__ bool idle(const SplitPlan& sp) const { return queued && (int)blockIdx.x >= sp.resident; }

  __device__ __forceinline__ bool first_thread() const { return wave == 0 && fresh_lane() == 0; }

  static __device__ __forceinline__ int32_t* counter(const SplitPlan& sp, int x) { return sp.queue + x * QUEUE_STRIDE; }

  // requests the number of the next item (the first one is the workgroup's own number: the counters start behind these)
  __device__ __forceinline__ void draw(const SplitPlan& sp) {
    if (!queued || out) return;
    out = true;
    if (first_thread()) drawn = __hip_atomic_fetch_add(counter(sp, xcd), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }

  // after an item: its number is known to all threads.  False: the launch is direct, there is no next one.
  __device__ __forceinline__ bool advance(const SplitPlan& sp) {
    if (!queued) return false;
    draw(sp);
    out = false;
    __syncthreads();                                     // (all threads are through with the LDS of this item)
    if (first_thread()) *word = drawn;
    drawn = 0;                                           // (no register is kept for it over the next item)
    __syncthreads();
    q = __builtin_amdgcn_readfirstlane(*word);
    return true;
  }

  // The item that number q of this XCD stands for; numbers without one (split units, the end of a chunk) are passed over.
  __device__ __forceinline__ bool take(WorkItem& it, const SplitPlan& sp, int units_per_head, int chunk, int heads,
                                       const int32_t* order) {
    it.part = 0; it.parts = 0; it.part_len = 0; it.slot = 0;
    auto part = [&](int g) {                             // part g of the plan's table
      const int32_t* pt = sp.part_table + 4 * g;
      const int unit = scalar_ld(pt);
      it.bh = unit / units_per_head; it.blk = unit % units_per_head;
      it.part = scalar_ld(pt + 1); it.parts = scalar_ld(pt + 2); it.part_len = scalar_ld(pt + 3);
      it.slot = g;
    };
    // position it.blk of the schedule -> block by the caller's launch order, then: is it one to walk whole?
    auto whole = [&]() -> bool {
      if (order) it.blk = min(max(scalar_ld(order + (int64_t)it.bh * units_per_head + it.blk), 0), units_per_head - 1);   // caller data
      return sp.pool_slots == 0 || scalar_ld(sp.unit_slot + (int64_t)it.bh * units_per_head + it.blk) < 0;
    };
    const int units = heads * units_per_head;
    auto in_stretch = [&](int x, int s) -> bool {        // place s of XCD x's stretch: `order` is the list of all of them
      const int at = stretch_first(units, x) + s;
      if (at >= stretch_first(units, x + 1)) return false;
      const int u = min(max(scalar_ld(order + at), 0), units - 1);
      it.bh = u / units_per_head; it.blk = u % units_per_head;
      return scalar_ld(sp.unit_slot + u) < 0;
    };
    if (!queued) {
      // parts first, whole columns right behind them (at a multiple of eight: the workgroup -> XCD phase stays).  The
      // host does not know the number of parts and launches room for the whole pool: what is too much comes last.
      // (Between the two it kept the columns of 24 heads of 21, 332 parts in front, waiting for 10 us: 51.7 / 49.1 us.)
      const int g = blockIdx.x, n = sp.pool_slots ? scalar_ld(sp.header) : 0, wg = g - ((n + 7) & ~7);
      if (g < n) {
        part(g);
        return true;
      }
      if (wg < 0) return false;
      // (eighths of unlike work: the stretches in turn, so that every XCD gets the same)
      if (sp.stretches) return in_stretch(scalar_ld(sp.header + 2) != 0 ? wg & 7 : stretch_in_turn(wg), wg >> 3);
      if (wg >= xcd_map_wgs(heads, units_per_head, chunk, SHORT_COLUMNS)) return false;
      const HeadBlock hb = xcd_map(wg, units_per_head, chunk, SHORT_COLUMNS);
      it.bh = hb.bh; it.blk = hb.blk;
      return hb.valid && whole();
    }
    const int n_parts = scalar_ld(sp.header), wgs = xcd_map_wgs(heads, units_per_head, chunk, SHORT_COLUMNS);
    auto share = [&](int x) -> int {
      return sp.stretches ? stretch_first(units, x + 1) - stretch_first(units, x) : xcd_map_share(wgs, x);
    };
    for (;;) {
      const int np = (n_parts - xcd + 7) >> 3;           // parts g = 8 q + xcd < n_parts
      if (q < np) {
        part(8 * q + xcd);
        return true;
      }
      const int s = q - np;
      if (s < share(xcd)) {
        if (sp.stretches) {
          if (in_stretch(xcd, s)) return true;
        } else {
          const HeadBlock hb = xcd_map(8 * s + xcd, units_per_head, chunk, SHORT_COLUMNS);
          it.bh = hb.bh; it.blk = hb.blk;
          if (hb.valid && whole()) return true;
        }
      } else {                                           // this XCD is through: on to the one with most items left
        __syncthreads();
        if (wave == 0) {
          const int x = fresh_lane() & 7;
          int left = share(x) + ((n_parts - x + 7) >> 3) -
                     __hip_atomic_load(counter(sp, x), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          left = left > 0 ? 8 * left + x : -1;
#pragma unroll
          for (int off = 4; off > 0; off >>= 1) left = max(left, __shfl_xor(left, off, 64));
          if (first_thread()) *word = left;
        }
        __syncthreads();
        const int at = __builtin_amdgcn_readfirstlane(*word);
        if (at < 0) return false;
        xcd = at & 7;
      }
      advance(sp);
    }
  }
};

// The kernel's (only) argument, read again from the argument segment: what a kernel that walks several items needs of
// it is then loaded anew per item instead of being kept in scalar registers, and spilled, across all of them.
template <typename Args>
__device__ __forceinline__ const Args& fresh_args() {
#if defined(__HIP_DEVICE_COMPILE__)
  auto p = (__attribute__((address_space(4))) const char*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const Args*)p;
#else
  return *(const Args*)nullptr;
#endif
}

}  // namespace spa2
