// The pattern listed per key block, and the order in which the dK/dV kernel takes the key blocks: as launches of their own
// (mask.hip), or as workgroups of launches that the backward pass makes anyway (split.hip, bwd.hip).
#pragma once
#include "spa2_device.h"
#include "spa2_internal.h"

namespace spa2 {

// One workgroup lists COLS key blocks of one head: thread (seg, c) takes one of SEGS runs of query blocks of column c,
// reads its mask bytes into one bit each (COL_BATCH loads in flight), and, after the counts of the column's runs have
// been exchanged through LDS, writes its ascending piece of the list at the right offset.  Runs of up to 64 query
// blocks (T_m <= 64 SEGS) stay in a register between the two steps; longer ones are read again, 64 at a time.
// Bound: load latency; a loop that read one byte at a time, twice, took 33 us for 4 heads of 1024 x 2048 blocks and 56 us
// for 40 of 591 x 1182; as a launch of its own, with 64 columns a workgroup, this takes 12 and 26 us.
constexpr int COL_BATCH = 16;
struct ColumnArgs {
  const uint8_t* mask; int32_t* col_cnt; int32_t* col_idx;
  int Tm, Tn, groups;          // groups of `cols` key blocks a head
};
inline ColumnArgs column_args(const uint8_t* mask, const Dims& m, int32_t* col_cnt, int32_t* col_idx, int cols) {
  return ColumnArgs{mask, col_cnt, col_idx, m.Tm, m.Tn, (m.Tn + cols - 1) / cols};
}
template <int SEGS, int COLS>
__device__ __forceinline__ void columns_block(const ColumnArgs& a, int bh, int group, int (&seg_cnt)[SEGS][COLS]) {
  const int Tm = a.Tm, Tn = a.Tn;
  const int c = threadIdx.x % COLS, seg = threadIdx.x / COLS;
  const int j = group * COLS + c;
  const int per = (Tm + SEGS - 1) / SEGS;
  const int i0 = min(Tm, seg * per), i1 = min(Tm, i0 + per);
  const bool live = j < Tn;
  const uint8_t* mp = a.mask + (int64_t)bh * Tm * Tn + min(j, Tn - 1);
  // bit x: query block i + x (below i1, 64 of them at most) selected this column
  auto bits_from = [&](int i) -> uint64_t {
    uint64_t bits = 0;
    for (int x0 = 0; x0 < 64 && i + x0 < i1; x0 += COL_BATCH) {
      uint8_t b[COL_BATCH];
#pragma unroll
      for (int x = 0; x < COL_BATCH; ++x) b[x] = mp[(int64_t)min(i + x0 + x, i1 - 1) * Tn];
#pragma unroll
      for (int x = 0; x < COL_BATCH; ++x) bits |= (uint64_t)(b[x] != 0 && i + x0 + x < i1 ? 1u : 0u) << (x0 + x);
    }
    return bits;
  };
  const uint64_t first = bits_from(i0);
  int n = __builtin_popcountll(first);
  for (int i = i0 + 64; i < i1; i += 64) n += __builtin_popcountll(bits_from(i));
  seg_cnt[seg][c] = n;
  __syncthreads();
  if (!live) return;
  int at = 0;
  for (int s2 = 0; s2 < seg; ++s2) at += seg_cnt[s2][c];
  int32_t* out = a.col_idx + ((int64_t)bh * Tn + j) * Tm;
  for (int i = i0; i < i1; i += 64) {
    uint64_t bits = i == i0 ? first : bits_from(i);
    while (bits) {
      out[at++] = i + __builtin_ctzll(bits);
      bits &= bits - 1;
    }
  }
  if (seg == SEGS - 1) a.col_cnt[(int64_t)bh * Tn + j] = at;
}

// Launch order of the key blocks of one head for the dK/dV kernel: longest column first (equal lengths: lower index
// first), dealt round-robin to the eight XCD chunks of the schedule (position x*chunk + s belongs to XCD x), so that
// every XCD gets the same mix of long and short columns and the long ones start early.  (Heads of up to SHORT_COLUMNS are
// launched position by position (xcd_map): there neighbouring positions, chunks of the order, are what mixes the lengths.)
// A column's rank is the number of columns that precede it in that order, counted directly: a workgroup ranks COLS
// columns of a head against all of them, SEGS threads a column, the head's keys in LDS.  (T_n^2 comparisons, but
// no chain of dependent steps: the bitonic sort of a head by one workgroup before took 11.6 us at 512 columns of 12
// heads and 23.6 us at 2048 columns of 4, this takes 4.8 and 5.5 us with the 1024 threads of a launch of its own.)
struct OrderArgs {
  const int32_t* col_cnt; int32_t* col_order;
  int Tn, groups;
};
inline OrderArgs order_args(const int32_t* col_cnt, const Dims& m, int32_t* col_order, int cols) {
  return OrderArgs{col_cnt, col_order, m.Tn, (m.Tn + cols - 1) / cols};
}
template <int NP, int SEGS, int COLS>
struct OrderLds {
  __attribute__((aligned(16))) uint32_t keys[NP];
  uint32_t before[SEGS][COLS];
};
template <int NP, int SEGS, int COLS>
__device__ __forceinline__ void order_block(const OrderArgs& a, int bh, int group, OrderLds<NP, SEGS, COLS>& lds) {
  const int Tn = a.Tn;
  auto &keys = lds.keys;
  auto &before = lds.before;
  const int tid = threadIdx.x, c = tid % COLS, seg = tid / COLS;
  const int padded = (Tn + 4 * SEGS - 1) / (4 * SEGS) * (4 * SEGS);      // (Tn <= NP: fits)
  const int per = padded / SEGS;                       // keys that one thread compares with, a multiple of four
  for (int j = tid; j < padded; j += COLS * SEGS)      // distinct keys: length, then lower index; padding below all
    keys[j] = j < Tn ? ((uint32_t)min(a.col_cnt[(int64_t)bh * Tn + j], 0xffff) << 16) | (uint32_t)(0xffff - j) : 0u;
  __syncthreads();
  const int j = group * COLS + c;
  const uint32_t mine = keys[min(j, Tn - 1)];
  uint32_t n = 0;
  for (int x = seg * per; x < min((seg + 1) * per, Tn); x += 4) {       // (a wave reads one address: broadcast)
    const u32x4 k4 = *(const u32x4*)(keys + x);
#pragma unroll
    for (int e = 0; e < 4; ++e) n += k4[e] > mine ? 1u : 0u;
  }
  before[seg][c] = n;
  __syncthreads();
  if (seg != 0 || j >= Tn) return;
  uint32_t rank = 0;
#pragma unroll
  for (int x = 0; x < SEGS; ++x) rank += before[x][c];
  // the schedule position that is dealt as number `rank`: rounds of all XCDs while the shortest chunk lasts, then of
  // those that still have positions (chunk x has min(chunk, T_n - x * chunk) of them)
  const int chunk = (Tn + 7) / 8;
  int left = (int)rank, s = 0, live = 8;
  while (live > 0) {
    const int len = min(max(Tn - (live - 1) * chunk, 0), chunk);        // the last live chunk is the shortest
    const int rounds = max(len - s, 0);
    if (left < rounds * live) break;
    left -= rounds * live;
    s += rounds;
    --live;
  }
  const int pos = (left % live) * chunk + s + left / live;
  a.col_order[(int64_t)bh * Tn + pos] = j;
}

// Launch order of the columns of all heads in stretches (stretch_first): place lo_x + s of the list is what XCD x takes as its
// s-th, a number bh * T_n + j.  One head after the other, longest column first, in long launches; longest first over the
// whole stretch (by_length) in launches of up to three rounds, whose last ones to start should be short.  Backward pass, us, by
// head / by length: 24 heads of 2000 tokens 66.7 / 62.3 (1.5 rounds), of 4000 132.7 / 121.3 (3), 32 heads of 8192, d = 64,
// (4) 576 / 587.  Ranks are counted, as above.
struct ListArgs {
  const int32_t* col_cnt; int32_t* list;
  int Tn, units, groups, by_length;          // groups of 64 columns a stretch
};
inline ListArgs list_args(const int32_t* col_cnt, const Dims& m, int32_t* list, bool by_length) {
  const int units = m.B * m.H * m.Tn;
  return ListArgs{col_cnt, list, m.Tn, units, ((units + 7) / 8 + 63) / 64, by_length};
}
struct ListLds {
  __attribute__((aligned(16))) uint32_t keys[SIDE_ORDER_MAX];
  uint32_t before[4][64];
};
__device__ __forceinline__ void list_block(const ListArgs& a, int xcd, int group, ListLds& lds) {
  const int lo = stretch_first(a.units, xcd), n = stretch_first(a.units, xcd + 1) - lo, h0 = lo / a.Tn;
  const int tid = threadIdx.x, c = tid & 63, seg = tid >> 6;
  const int padded = (n + 15) & ~15, per = padded / 4;
  // distinct keys: (lower head,) length (T_m < 512), lower number; padding below all
  for (int s = tid; s < padded; s += 256) {
    const uint32_t len = s < n ? (uint32_t)min(max(a.col_cnt[lo + s], 0), 511) : 0u;
    const uint32_t head = a.by_length ? 0u : (uint32_t)(2047 - min((lo + s) / a.Tn - h0, 2047));
    lds.keys[s] = s < n ? (head << 21) | (len << 12) | (uint32_t)(4095 - s) : 0u;
  }
  __syncthreads();
  const int s = group * 64 + c;
  const uint32_t mine = lds.keys[min(s, max(n - 1, 0))];
  uint32_t before = 0;
  for (int x = seg * per; x < (seg + 1) * per; x += 4) {       // (a wave reads one address: broadcast)
    const u32x4 k4 = *(const u32x4*)(lds.keys + x);
#pragma unroll
    for (int e = 0; e < 4; ++e) before += k4[e] > mine ? 1u : 0u;
  }
  lds.before[seg][c] = before;
  __syncthreads();
  if (seg != 0 || s >= n) return;
  a.list[lo + (int)(lds.before[0][c] + lds.before[1][c] + lds.before[2][c] + lds.before[3][c])] = lo + s;
}

}  // namespace spa2
