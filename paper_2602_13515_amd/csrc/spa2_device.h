// Device-side helpers shared by the spa2 kernels (gfx950 / CDNA4, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace spa2 {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

// address-space qualified pointers of the direct global -> LDS copy builtin
typedef __attribute__((address_space(1))) const void gptr_t;
typedef __attribute__((address_space(3))) void lptr_t;

constexpr int BQ = 128;
constexpr int BKV = 64;
constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;

// Operand layout of the bf16 MFMA shape used here (lane l of a wave64):
//   32x32x16:  A[m][k]: m = l%32, k = 8*(l/32)+s (s=0..7)   B[k][n]: n = l%32, same k
//              C[m][n]: n = l%32, m = 8*(v/4) + 4*(l/32) + v%4 for accumulator register v = 0..15
__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// compile-time loop: f(Int<B>{}), ..., f(Int<E-1>{})
template <int I> struct Int { static constexpr int v = I; };
template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) { f(Int<B>{}); static_for<B + 1, E>(f); }
}

// Two floats -> packed bf16 pair (round to nearest even), low half = a.
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  f32x2 v = {a, b};
  bf16x2 r = __builtin_convertvector(v, bf16x2);
  return __builtin_bit_cast(uint32_t, r);
}

// Transposing LDS read (ds_read_b64_tr_b16).  Within each group of 16 lanes,
// lane s supplies the address of four consecutive 16-bit elements; lane i of
// the group receives element (i%4) of the data addressed by lanes i/4, 4+i/4,
// 8+i/4, 12+i/4.  If lane s points at row (s/4), columns 4*(s%4).. of a
// row-major tile, lane i ends up with column i of rows 0..3: a 4x16 patch read
// column-wise, which is what an MFMA operand needs when the contraction index
// is the row of the tile in memory.
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
__device__ __forceinline__ bf16x8 join_tr(u32x2 lo, u32x2 hi) {
  u32x4 u = {lo[0], lo[1], hi[0], hi[1]};
  return __builtin_bit_cast(bf16x8, u);
}

// Exchange between the two 32-lane halves of a wave on the vector ALU (v_permlane32_swap), without a trip
// through LDS: max / sum of the values that lanes l and l^32 hold, in both lanes.
__device__ __forceinline__ void both_halves(float x, float& lo, float& hi) {
  const uint32_t u = __builtin_bit_cast(uint32_t, x);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  lo = __builtin_bit_cast(float, (uint32_t)r[0]);
  hi = __builtin_bit_cast(float, (uint32_t)r[1]);
}
__device__ __forceinline__ float max_halves(float x) { float lo, hi; both_halves(x, lo, hi); return fmaxf(lo, hi); }
__device__ __forceinline__ float sum_halves(float x) { float lo, hi; both_halves(x, lo, hi); return lo + hi; }

// acc + lo(p) + hi(p) for a packed bf16 pair p, accumulated in fp32 (v_dot2c_f32_bf16 with a pair of ones)
__device__ __forceinline__ float dot2_ones(uint32_t p, float acc) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, p), __builtin_bit_cast(bf16x2, 0x3f803f80u), acc,
                                         false);
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ void raw_copies_done() {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#endif
}
// All but the last COUNT vector-memory operations of the wave are done (they complete in order).
template <int COUNT>
__device__ __forceinline__ void raw_copies_left() {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_waitcnt vmcnt(%0)" :: "n"(COUNT) : "memory");
#endif
}

// A number that an earlier launch has written, at a uniform address: as a scalar load (the compiler makes a vector load of it
// where the kernel may write through another pointer).
__device__ __forceinline__ int scalar_ld(const int32_t* p) {
#if defined(__HIP_DEVICE_COMPILE__)
  return *(__attribute__((address_space(4))) const int32_t*)p;
#else
  return *p;
#endif
}

// Everything above has been requested here: loads are not moved down behind the branches that follow.
__device__ __forceinline__ void requested() {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" ::: "memory");
#endif
}

// Entry `at` of an index list into a register, waited for here: a load inside a branch that is first used behind it would
// make the compiler wait for every outstanding memory operation there, copies included, also where the branch is not taken.
__device__ __forceinline__ int list_load(const int32_t* idx, int at) {
  int x = idx[at];
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(x));
#endif
  return x;
}

// LDS accesses by 32-bit byte address.  A generic pointer into LDS is turned into its LDS address once
// (lds_addr_of); from then on addresses are plain integers, so that address arithmetic stays 32-bit and constant
// parts can be folded into the instructions' offset fields, and no generic-pointer null checks are generated.
typedef __attribute__((address_space(3))) const bf16x8 lds_cbf16x8;
typedef __attribute__((address_space(3))) const f32x4 lds_cf32x4;
typedef __attribute__((address_space(3))) float lds_f32;
typedef __attribute__((address_space(3))) u32x2 lds_u32x2;
typedef __attribute__((address_space(3))) const u32x4 lds_cu32x4;
__device__ __forceinline__ uint32_t lds_addr_of(const void* p) { return (uint32_t)(size_t)(lptr_t*)p; }
#if defined(__HIP_DEVICE_COMPILE__)      // (LDS pointers are 32 bits wide only in the device pass)
__device__ __forceinline__ bf16x8 lds_ld16(uint32_t addr) { return *(lds_cbf16x8*)addr; }
__device__ __forceinline__ f32x4 lds_ldf4(uint32_t addr) { return *(lds_cf32x4*)addr; }
__device__ __forceinline__ void lds_stf(uint32_t addr, float x) { *(lds_f32*)addr = x; }
__device__ __forceinline__ void lds_st8(uint32_t addr, u32x2 x) { *(lds_u32x2*)addr = x; }
__device__ __forceinline__ u32x4 lds_ldu4(uint32_t addr) { return *(lds_cu32x4*)addr; }
__device__ __forceinline__ u32x2 lds_tr4_at(uint32_t addr) {
  s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)addr);
  return __builtin_bit_cast(u32x2, v);
}
#else
__device__ bf16x8 lds_ld16(uint32_t addr);
__device__ f32x4 lds_ldf4(uint32_t addr);
__device__ void lds_stf(uint32_t addr, float x);
__device__ void lds_st8(uint32_t addr, u32x2 x);
__device__ u32x4 lds_ldu4(uint32_t addr);
__device__ u32x2 lds_tr4_at(uint32_t addr);
#endif
// Direct global -> LDS copy, 16 bytes per lane: lane l's bytes land at lds_addr + LDS_CONST + 16 l (lds_addr wave-uniform);
// the source is a wave-uniform base plus a 32-bit byte offset per lane.  Issued as an assembly statement so
// that the compiler's wait-count insertion does not see it: through the builtin, LDS reads that follow a copy
// are made to wait for it (the two cannot be told apart by address).  The caller therefore owns the
// ordering: raw_copies_done() before the barrier that publishes the tile.  In-order completion of vector
// memory operations keeps the compiler's own counted waits safe (they can only wait for more, never less).
// m0 carries the LDS address and is declared clobbered; a kernel that uses this helper must not also rely on
// the compiler keeping a value of its own in m0 across it (the builtin form of the same copy would).
// LDS_CONST is a compile-time part of the destination that is added while m0 is written.
template <int LDS_CONST>
__device__ __forceinline__ void raw_copy16_to_lds_at(const void* src_base, uint32_t src_off, uint32_t lds_addr) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :: "s"(lds_addr), "v"(src_off), "s"(src_base), "n"(LDS_CONST) : "memory", "m0", "scc");
#endif
}
template <int LDS_CONST>
__device__ __forceinline__ void raw_copy4_to_lds_at(const void* src_base, uint32_t src_off, uint32_t lds_addr) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2"
               :: "s"(lds_addr), "v"(src_off), "s"(src_base), "n"(LDS_CONST) : "memory", "m0", "scc");
#endif
}

// XOR-swizzled LDS tile: rows of D bf16, unpadded; the 16-byte chunk c of row r lives at chunk position
// c ^ swz<D>(r).  The function is chosen so that BOTH access patterns the kernels use are free of bank
// conflicts (64 banks x 4 bytes): 16 lanes reading the same chunk of 16 consecutive rows (MFMA operand read
// along rows), and 32 lanes reading 64 contiguous bytes of each of 4 consecutive rows (transposing read).
template <int D> __device__ __forceinline__ int swz(int r);
template <> __device__ __forceinline__ int swz<128>(int r) { return ((r & 3) << 2) | ((r >> 2) & 3); }
template <> __device__ __forceinline__ int swz<64>(int r) { return (((r >> 1) & 1) << 2) | ((r >> 2) & 3); }
// element index of logical (row, col) in a swizzled tile
template <int D> __device__ __forceinline__ int swz_idx(int row, int col) {
  return row * D + ((((col >> 3) ^ swz<D>(row))) << 3) + (col & 7);
}

// ---- results on their way out.  In the accumulators a lane owns one token row and eight bytes of it at a time, so that a
// store straight from there touches 32 rows and 16 bytes of each.  The 32 rows of a wave therefore go through 32 * D * 2
// bytes of LDS (`area`, the wave's own) and are stored as whole rows, 16 bytes a lane.  Chunk c (16 bytes) of row r lies at
// chunk position c ^ (r % (D / 8)): lanes of neighbouring rows write to different banks.
// Measured, us a call, stores from the accumulators / this: 4 samples of 1281 tokens, 6 heads, forward and backward 116.4 /
// 109.3; 20,010 tokens, 6 heads, d = 64 314 / 306; 32,760 tokens, 12 heads 1985 / 1939; 75,600 tokens, 40 heads, forward 4310 /
// 4202 (same bits).
template <int D>
__device__ __forceinline__ void row_piece_put(uint32_t area, int row, int chunk, int half, u32x2 x) {
  lds_st8(area + row * (D * 2) + ((chunk ^ (row & (D / 8 - 1))) << 4) + 8 * half, x);
}
// the first `valid` of the wave's rows to dst (row 0), sn elements apart
template <int D>
__device__ __forceinline__ void rows_store(uint32_t area, uint16_t* dst, int64_t sn, int valid, int lane) {
  constexpr int CPR = D / 8, RPI = 64 / CPR;         // chunks per row, rows per instruction
  const int c = lane % CPR, r0 = lane / CPR;
#pragma unroll
  for (int r = 0; r < 32; r += RPI) {
    const int row = r + r0;
    const u32x4 x = lds_ldu4(area + row * (D * 2) + ((c ^ (row & (CPR - 1))) << 4));
    if (row < valid) *(u32x4*)(dst + row * sn + 8 * c) = x;
  }
}

// ---- partial results of split lists (split.hip), handed from one workgroup to another inside a launch.  The two may
// run on different XCDs, whose L2 caches are not coherent with each other: partial results are therefore written and
// read with device-scope atomic accesses (write-through / L2-bypassing, 8 bytes a lane), which need no cache
// write-back or invalidation around the hand-over.  Plain 16-byte accesses with a device-scope fence instead (one L2
// write-back per part) took 205 against 162 us for dK/dV on a 20,010-token, 6-head, d = 64 layer.
__device__ __forceinline__ void part_store2(float* p, float x, float y) {
  const f32x2 v = {x, y};
  __hip_atomic_store((uint64_t*)p, __builtin_bit_cast(uint64_t, v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ f32x2 part_load2(const float* p) {
  return __builtin_bit_cast(f32x2, __hip_atomic_load((const uint64_t*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}
// Counts the calling workgroup's part in (all of its threads call this after their part_store2) and says whether it
// was the last of `parts`.  lds_word: any LDS word that is free at this point.
__device__ __forceinline__ bool last_part(int32_t* arrive, int parts, int* lds_word) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // this wave's stores have reached the coherence point
#endif
  __syncthreads();                                     // ... and so have those of the other waves
  if (threadIdx.x == 0) *lds_word = __hip_atomic_fetch_add(arrive, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  return *lds_word == parts - 1;
}

// Workgroup id -> (head, block) mapping that keeps one head's blocks resident on all eight XCDs at once: consecutive
// workgroup ids go round-robin to the XCDs, so XCD x receives ids x, x+8, ...; those are given a contiguous chunk of the
// head's blocks, which share K/V tiles through that XCD's L2.  The last chunk is a short one and, where blocks are dealt to
// the chunks by length, the first holds the longest, which counts in heads of few blocks: up to MIDDLE_HEAD every head
// starts with another XCD, and up to SHORT_ROWS or SHORT_COLUMNS, where a chunk is a few blocks and the last ones are empty,
// the blocks go to the XCDs in turn instead.
// Measured, us, chunk x always on XCD x / now (forward, dQ, dK/dV; d = 128 unless noted).  In turn: 11 rows and 21 columns,
// 24 heads 32.2 / 30.7, 31.2 / 30.1, 53.0 / 50.3; the same, d = 64, 512 heads 156 / 117, 148 / 111, (drawn from a queue).
// Another XCD: 65 rows, 40 heads 185 / 176, 196 / 184; 97 rows, 24 heads, d = 64 105 / 102, 116 / 114; on longer heads it
// gives nothing (157 rows) and loses 1 % of the forward pass on 591.
// The line between the two, us, chunks that start with another XCD / in turn.  Forward: 20 rows, 24 heads 36.0 / 30.0; 31 rows
// 54.8 / 53.5; 32 rows, whose chunks are even, 12 heads 33.0 / 35.2, 40 heads, d = 64 45 / 49, over 48 launches of 12 to 64 heads
// 1 % faster in chunks (dQ the same); even chunks of 1 to 3 rows -2 to +2 %.  dK/dV: 25 columns, 76 heads 141 / 114; 31 columns
// 147 / 126; 32 columns, 60 heads 143 / 123 (few long columns: the chunks' first positions); 79 columns, 12 heads 62 / 65.
struct HeadBlock { int bh; int blk; bool valid; };
constexpr int SHORT_ROWS = 31, SHORT_COLUMNS = 32, MIDDLE_HEAD = 128;
// number of workgroups that xcd_map deals the blocks of all heads to (short_head: SHORT_ROWS or SHORT_COLUMNS)
__host__ __device__ __forceinline__ int xcd_map_wgs(int heads, int blocks_per_head, int chunk, int short_head) {
  return heads * (blocks_per_head <= short_head ? blocks_per_head : 8 * chunk);
}
// ... and how many of them are dealt to XCD x: numbers x, x + 8, x + 16, ...
__host__ __device__ __forceinline__ int xcd_map_share(int wgs, int xcd) { return (wgs - xcd + 7) >> 3; }
__host__ __device__ __forceinline__ HeadBlock xcd_map(int wg, int blocks_per_head, int chunk, int short_head) {
  HeadBlock r;
  if (blocks_per_head <= short_head) {
    r.bh = wg / blocks_per_head;
    r.blk = (wg - r.bh * blocks_per_head + 3 * r.bh) % blocks_per_head;
    r.valid = true;
    return r;
  }
  const int xcd = wg & 7;
  const int slot = wg >> 3;
  r.bh = slot / chunk;
  r.blk = ((xcd + (blocks_per_head <= MIDDLE_HEAD ? 3 * r.bh : 0)) & 7) * chunk + slot % chunk;
  r.valid = r.blk < blocks_per_head;
  return r;
}

// The same for rows, which are launched in the order of the sequence: every four consecutive rows of an XCD are
// rotated by a hash of their number.  Workgroups of an XCD are handed to its shader engines in turn and in order, and
// an engine that is full holds back the ones behind it; rows whose lengths alternate (long, short, long, short: 256 and
// 55 tiles on 32,768 tokens, 24 heads) otherwise put all long ones on the same engines.  Measured there: forward
// 5438 -> 4526 us, dQ 7847 -> 6310 us; rows without such a structure (75,600 tokens, 40 heads) 7665 -> 7607 and
// 10498 -> 10589 us.  A queue that 512 resident workgroups draw rows from evens out as much, but costs 3 us a row: 4 %
// on rows of 36 tiles.
__host__ __device__ __forceinline__ HeadBlock xcd_map_rows(int wg, int blocks_per_head, int chunk) {
  HeadBlock r = xcd_map(wg, blocks_per_head, chunk, SHORT_ROWS);
  const int s = (wg >> 3) % chunk;
  if (blocks_per_head > SHORT_ROWS && (s | 3) < chunk) {    // (the last rows of a chunk that fill no group of four stay in place)
    const uint32_t rot = ((uint32_t)r.bh * 0x85EBCA6Bu + (uint32_t)(s >> 2) * 0x9E3779B1u) >> 30;   // one per group
    const int t = (s & ~3) | ((s + (int)rot) & 3);
    r.blk += t - s;
    r.valid = r.blk < blocks_per_head;
  }
  return r;
}

// Rotation inside groups of four, as above, of place s of an XCD's stretch of n rows.
__host__ __device__ __forceinline__ int rotated_row(int s, int n, int xcd) {
  if ((s | 3) >= n) return s;
  const uint32_t rot = ((uint32_t)xcd * 0x85EBCA6Bu + (uint32_t)(s >> 2) * 0x9E3779B1u) >> 30;
  return (s & ~3) | ((s + (int)rot) & 3);
}
// Rows (or columns) in stretches, an eighth of all of them for each XCD, one head after the other (with_stretches).
__host__ __device__ __forceinline__ int stretch_first(int units, int xcd) { return (int)((int64_t)units * xcd >> 3); }
__host__ __device__ __forceinline__ int stretch_wgs(int units) { return (units + 7) & ~7; }
// The stretch that workgroup wg takes its place wg >> 3 of, where the XCDs take the stretches in turn.
__host__ __device__ __forceinline__ int stretch_in_turn(int wg) { return (wg + (wg >> 3)) & 7; }
__host__ __device__ __forceinline__ HeadBlock stretch_row(int wg, int heads, int blocks_per_head) {
  const int units = heads * blocks_per_head, x = wg & 7, s = wg >> 3;
  const int lo = stretch_first(units, x), n = stretch_first(units, x + 1) - lo;
  const int u = lo + rotated_row(s, n, x);
  return HeadBlock{u / blocks_per_head, u % blocks_per_head, s < n};
}

}  // namespace spa2
