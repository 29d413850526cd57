// D = rowsum(dO * (O + o_res)), the one quantity both backward kernels need per query row.
// Bound: HBM (three bf16 tensors read once, 302 MB in 60 us on the 32,760-token, 12-head layer: 5.0 TB/s, what a large
// device copy reaches).  All loads of a workgroup are issued before the first use.
#pragma once
#include "spa2_device.h"
#include "spa2_internal.h"

namespace spa2 {

struct DeltaArgs {
  const uint16_t* o; const uint16_t* o_res; const uint16_t* d_o; float* delta;
  int H, N, chunks; int64_t sb, sh, sn;
};

constexpr int DELTA_NIT = 4;          // row groups per workgroup
inline int delta_rows_per_wg(int d) { return DELTA_NIT * 256 / (d / 8); }

template <int D>
__device__ __forceinline__ void delta_block(const DeltaArgs& a, int bh, int chunk) {
  constexpr int LPR = D / 8, RP = 256 / LPR, NIT = DELTA_NIT;
  const int64_t base = (int64_t)(bh / a.H) * a.sb + (int64_t)(bh % a.H) * a.sh;
  const int tid = threadIdx.x;
  const int col = (tid % LPR) * 8;
  u32x4 x[NIT], y[NIT], z[NIT];
  int row[NIT];
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    row[it] = (chunk * NIT + it) * RP + tid / LPR;
    const int64_t off = base + (int64_t)min(row[it], a.N - 1) * a.sn + col;   // rows past the end: clamped, not stored
    x[it] = *(const u32x4*)(a.o + off);
    y[it] = *(const u32x4*)(a.d_o + off);
    z[it] = u32x4{0, 0, 0, 0};
  }
  if (a.o_res) {
#pragma unroll
    for (int it = 0; it < NIT; ++it)
      z[it] = *(const u32x4*)(a.o_res + base + (int64_t)min(row[it], a.N - 1) * a.sn + col);
  }
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    float s = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float o0 = __builtin_bit_cast(float, x[it][e] << 16) + __builtin_bit_cast(float, z[it][e] << 16);
      const float o1 = __builtin_bit_cast(float, x[it][e] & 0xffff0000u) + __builtin_bit_cast(float, z[it][e] & 0xffff0000u);
      s = fmaf(o0, __builtin_bit_cast(float, y[it][e] << 16), s);
      s = fmaf(o1, __builtin_bit_cast(float, y[it][e] & 0xffff0000u), s);
    }
#pragma unroll
    for (int off = LPR / 2; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if (row[it] < a.N && (tid % LPR) == 0) a.delta[(int64_t)bh * a.N + row[it]] = s;
  }
}

inline DeltaArgs delta_args(const void* o, const void* o_res, const void* d_o, const Dims& m, float* delta) {
  DeltaArgs a;
  a.o = (const uint16_t*)o; a.o_res = (const uint16_t*)o_res; a.d_o = (const uint16_t*)d_o; a.delta = delta;
  a.H = m.H; a.N = m.N; a.sb = m.sb; a.sh = m.sh; a.sn = m.sn;
  const int rows = delta_rows_per_wg(m.d);
  a.chunks = (m.N + rows - 1) / rows;
  return a;
}

}  // namespace spa2
