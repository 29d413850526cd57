// Block-sparse attention backward for gfx950 (gradients of Alg. 1's O w.r.t. Q, K, V with
// the block mask held constant; Sec. 4.3 only states that a backward pass exists, the
// formulas are the usual softmax-attention calculus):
//   P = exp(S - LSE) on selected tiles,  dV = P^T dO,  dP = dO V^T,  D = rowsum(dO * O),
//   dS = P * (dP - D),  dQ = dS K * scale,  dK = dS^T Q * scale.
//
//   delta_kernel  D, one pass over O and dO (as a stage call; spa2_bwd makes the split plans in the same launch, see
//                 bwd_prepare_kernel in split.hip).
//   dq_kernel     one workgroup per query block, walking its row of the mask (same shape
//                 as the forward kernel: a lane owns one query row).
//   dkdv_kernel   one workgroup per key block, walking the query blocks that selected it.
// dQ is produced by a second, row-oriented pass instead of atomics: results are
// deterministic and there is no fp32 dQ scratch tensor.
#include "columns.h"
#include "row_delta.h"
#include "row_map.h"
#include "spa2_device.h"
#include "spa2_internal.h"
#include "split_plan.h"

namespace spa2 {

// ------------------------------------------------------------------ D = rowsum(dO * O)
template <int D>
__global__ __launch_bounds__(256) void delta_kernel(DeltaArgs a) { delta_block<D>(a, blockIdx.y, blockIdx.x); }

hipError_t launch_bwd_delta(const void* o, const void* o_res, const void* d_o, const Dims& m, float* delta,
                            hipStream_t stream) {
  const DeltaArgs a = delta_args(o, o_res, d_o, m, delta);
  const dim3 grid((unsigned)a.chunks, (unsigned)(m.B * m.H)), block(256);
  if (m.d == 128) hipLaunchKernelGGL(delta_kernel<128>, grid, block, 0, stream, a);
  else            hipLaunchKernelGGL(delta_kernel<64>, grid, block, 0, stream, a);
  return hipGetLastError();
}

// ------------------------------------------------------------------ dQ
struct DqArgs {
  const uint16_t* q; const uint16_t* k; const uint16_t* v; const uint16_t* d_o;
  const float* lse; const float* delta; uint16_t* dq;
  const int32_t* row_cnt; const int32_t* row_idx; const int32_t* row_order;
  int BH, H, N, Tm, Tn, chunk;
  int64_t sb, sh, sn;
  float scale, scale_log2;
  SplitPlan sp;         // long rows cut into parts (split.hip); sp.pool_slots == 0: every row is walked whole
  // What the dK/dV kernel needs of the column lists, made by workgroups of this launch: its plan by the first of `front`
  // in front of the parts (a multiple of eight: the workgroup -> XCD phase stays), its launch order by `orders` at the end.
  PlanArgs col_plan;
  OrderArgs col_order; ListArgs col_list;        // (one of them, by whether the launch is in stretches)
  int front, orders;
  bool stretches;
};

// Partial result of one part of a split row: the fp32 accumulators as [pair of registers][thread] (see fwd.hip).
template <int D> constexpr int dq_slot_floats() { return 256 * (D / 2); }
size_t dq_slot_bytes(const Dims& m) { return (size_t)(m.d == 128 ? dq_slot_floats<128>() : dq_slot_floats<64>()) * 4; }

// dQ = acc * scale -> bf16; a lane owns one query row, accumulator register v of block mb is channel
// 32 mb + 8 (v / 4) + 4 hf + v % 4.
template <int D>
__device__ __forceinline__ void dq_store_rows(const DqArgs& a, int64_t base, int q0, int lane, uint32_t area,
                                              const f32x16 (&acc)[D / 32]) {
  __syncthreads();          // (other waves may still be reading what lies in `area`)
#pragma unroll
  for (int mb = 0; mb < D / 32; ++mb)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      u32x2 pk = {pack_bf16(acc[mb][4 * g + 0] * a.scale, acc[mb][4 * g + 1] * a.scale),
                  pack_bf16(acc[mb][4 * g + 2] * a.scale, acc[mb][4 * g + 3] * a.scale)};
      row_piece_put<D>(area, lane & 31, 4 * mb + g, lane >> 5, pk);
    }
  rows_store<D>(area, a.dq + base + (int64_t)q0 * a.sn, a.sn, min(32, a.N - q0), lane);
}

// Transposed formulation, a lane owns one query row (see fwd.hip):
//   S^T  = K_j Q_i^T        P^T  = exp(S^T - LSE)
//   dP^T = V_j dO_i^T       dS^T = P^T * (dP^T - D)
//   dQ^T += K_j^T dS^T      (K^T through transposing LDS reads)
// The key block is taken in halves of 32 keys: S, dP of half 0, S, dP of half 1, then dQ of both.  The exponentials of a
// half run between its dP products and its dS between the products after those, and dP starts from -D, held in registers
// as a first accumulator, so dS costs one multiplication an element.
// Bound: the board's power (1.54 GHz) with the matrix cores busy 78 % of the cycles: 3960 cycles a tile and wave at two
// waves per SIMD for 1536 of matrix products (5200 before, when the mask of a short last block was worked out for every
// tile, 128 of 336 vector instructions, the copies multiplied out their offsets, and all exponentials stood in one run).
// Measured, us, before / after: 75,600 tokens, 40 heads 10877 / 9674; 32,760 tokens, 12 heads 662 / 574; 32,768 tokens,
// 24 heads, half the rows long 6466 / 5435; 20,010 tokens, 6 heads, d = 64 89 / 78.
template <int D>
__global__ __launch_bounds__(256, 2) void dq_kernel(DqArgs a) {
  constexpr int NK = D / 16, NMB = D / 32;           // contraction steps of S and dP, output blocks of dQ
  // K and V tiles, XOR-swizzled and unpadded (the layout a direct global -> LDS copy can write): K is read along rows
  // (S^T) and transposed (dQ^T), V along rows (dP^T).  (Aligned: compile-time parts are XORed into addresses.)
  constexpr int TILE_B = BKV * D * 2, STAGE_B = 2 * TILE_B;
  __shared__ __align__(1024) unsigned char smem[2 * STAGE_B];   // stage s: K tile, then V tile
  static_assert(sizeof(PlanLds<256>) <= 2 * STAGE_B && sizeof(OrderLds<SIDE_ORDER_MAX, 4, 64>) <= 2 * STAGE_B &&
                sizeof(ListLds) <= 2 * STAGE_B, "other work fits the tiles' LDS");

  // Which row, and which part of its list (see fwd.hip: the first sp.pool_slots workgroups are the parts of split rows)
  int bh, i, part = 0, parts = 0, part_len = 0;
  bool whole = false;
  const int slot = (int)blockIdx.x - a.front;
  if (slot < 0) {
    if (blockIdx.x == 0) plan_block<256>(a.col_plan, *(PlanLds<256>*)smem);
    return;
  }
  if ((int)blockIdx.x >= (int)gridDim.x - a.orders) {
    const int o = (int)blockIdx.x - ((int)gridDim.x - a.orders);
    if (a.stretches) list_block(a.col_list, o / a.col_list.groups, o % a.col_list.groups, *(ListLds*)smem);
    else order_block(a.col_order, o / a.col_order.groups, o % a.col_order.groups, *(OrderLds<SIDE_ORDER_MAX, 4, 64>*)smem);
    return;
  }
  if (slot < a.sp.pool_slots) {
    if (slot >= scalar_ld(a.sp.header)) return;
    const int32_t* pt = a.sp.part_table + 4 * slot;
    const int unit = scalar_ld(pt);
    part = scalar_ld(pt + 1); parts = scalar_ld(pt + 2); part_len = scalar_ld(pt + 3);
    bh = unit / a.Tm; i = unit % a.Tm;
  } else {
    const int wg = slot - a.sp.pool_slots;
    const HeadBlock hb = launched_row(a.sp, wg, a.BH, a.Tm, a.chunk);
    if (!hb.valid) return;
    bh = hb.bh;
    i = a.row_order ? min(max(a.row_order[(int64_t)bh * a.Tm + hb.blk], 0), a.Tm - 1) : hb.blk;
    whole = a.sp.pool_slots != 0;
  }
  const int64_t base = (int64_t)(bh / a.H) * a.sb + (int64_t)(bh % a.H) * a.sh;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);     // wave-uniform, in a scalar register
  const int r32 = lane & 31, hf = lane >> 5;
  const int N = a.N;
  const int64_t unit = (int64_t)bh * a.Tm + i;
  int cnt = min(max(a.row_cnt[unit], 0), a.Tn);   // clamped: see fwd.hip
  const int split_at = *(whole ? a.sp.unit_slot + unit : a.row_cnt + unit);
  const int first = part * part_len;         // entries [first, first + part_len) of the list of a split row
  const int32_t* idx = a.row_idx + unit * a.Tn + first;
  // the index list, 64 entries at a time in one register (lane l holds entry 64c + l): reading an entry is
  // a lane read, not a memory access whose result the loop would have to wait for.  (The first ones and the rows are
  // requested before the count is known: see fwd.hip.)
  int idx_v = idx[min(lane, a.Tn - 1 - first)];
  const int qrow = i * BQ + w * 32 + r32;
  const int qrow_ld = qrow < N ? qrow : N - 1;
  bf16x8 qf[D / 16], dof[D / 16];
  {
    const int64_t off = base + (int64_t)qrow_ld * a.sn + 8 * hf;
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) {
      qf[kk] = *(const bf16x8*)(a.q + off + 16 * kk);
      dof[kk] = *(const bf16x8*)(a.d_o + off + 16 * kk);
    }
  }
  const float lse2 = a.lse[(int64_t)bh * N + qrow_ld] * LOG2E;
  const float dlt = a.delta[(int64_t)bh * N + qrow_ld];
  requested();
  if (whole && split_at >= 0) return;
  if (parts) cnt = min(cnt - first, part_len);

  if (cnt == 0) {
    if (qrow < N) {
      uint16_t* op = a.dq + base + (int64_t)qrow * a.sn + (D / 2) * hf;
#pragma unroll
      for (int c = 0; c < D / 16; ++c) *(u32x4*)(op + 8 * c) = u32x4{0, 0, 0, 0};
    }
    return;
  }

  // K/V tiles are copied global -> LDS directly (no staging registers).  The destination of a wave-wide
  // 16-byte-per-lane copy is linear (wave base + 16 * lane), so the swizzle is applied on the source side: the
  // lane that fills chunk position pc of a row fetches logical chunk pc ^ swz(row).  Thread t fills chunk
  // position t % CPR of rows t / CPR + r * RSTEP; RSTEP is a multiple of 16 rows, so the swizzle term is the
  // same for every r.  Rows past N (short last block) are clamped to the last token (their P is made zero); the lane
  // offsets are computed again only when the number of valid rows changes.
  constexpr int CPR = D / 8, RSTEP = 256 / CPR, CH = BKV / RSTEP;
  // (what the rare paths of the loop need of the thread's number is worked out there, from the number itself: held in
  // registers over the loop it would cost spills)
  auto fresh_tid = [&]() -> int {
    int t = tid;
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+v"(t));
#endif
    return t;
  };
  uint32_t voff[CH];
  int rows_set = -1;
  auto set_rows = [&](int last) {            // last: last valid row of the tile (uniform)
    if (last == rows_set) return;
    rows_set = last;
    const int t = fresh_tid(), ld_row = t / CPR, ld_c8 = ((t % CPR) ^ swz<D>(ld_row)) * 8;
#pragma unroll
    for (int r = 0; r < CH; ++r) voff[r] = (uint32_t)((min(ld_row + RSTEP * r, last) * a.sn + ld_c8) * 2);
  };
  const uint32_t sm = lds_addr_of(smem);
  const char* k_head = (const char*)(a.k + base);
  const char* v_head = (const char*)(a.v + base);
  const uint64_t tile_bytes = (uint64_t)a.sn * (2 * BKV);
  constexpr int NPIECE = 2 * CH;             // piece p of a tile's copies: rows p / 2 of K (p even) or V
  auto copy_piece = [&](auto P, const char* kp, const char* vp, uint32_t stage) {
    constexpr int p = decltype(P)::v, r = p >> 1;
    raw_copy16_to_lds_at<(p & 1) * TILE_B + r * 4096>((p & 1) ? vp : kp, voff[r], stage + w * 1024);
  };

  f32x16 acc[NMB];
#pragma unroll
  for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[mb][v] = 0.f;
  f32x16 neg_d;                              // -D of this lane's query: the initial value of dP
#pragma unroll
  for (int v = 0; v < 16; ++v) neg_d[v] = -dlt;

  // per-lane LDS byte offsets inside a stage.  K row reads: row 32kb + r32, logical chunk 2kk + hf; the part of the
  // chunk index that depends on kk is XORed in as (kk << 5); the V row reads use the same offsets.
  // K transposing reads: rows (16-row group) + 8*which + 4hf + (s16>>2), columns 32mb + 16hb + 4(s16&3);
  // the part that depends on mb is XORed in as (mb << 6)
  const int s16 = lane & 15, hb16 = (lane >> 4) & 1;
  const uint32_t ka_off = sm + 2 * swz_idx<D>(r32, 8 * hf);
  const uint32_t kt_off0 = sm + 2 * swz_idx<D>(4 * hf + (s16 >> 2), 16 * hb16 + 4 * (s16 & 3));
  const uint32_t kt_off1 = sm + 2 * swz_idx<D>(8 + 4 * hf + (s16 >> 2), 16 * hb16 + 4 * (s16 & 3));

  auto list_entry = [&](int t) -> int {      // t uniform, inside the chunk that idx_v holds
    return min(max(__builtin_amdgcn_readlane(idx_v, t & 63), 0), a.Tn - 1);
  };
  int j_cur = list_entry(0);
  set_rows(min(BKV - 1, N - 1 - j_cur * BKV));
  static_for<0, NPIECE>([&](auto P) { copy_piece(P, k_head + j_cur * tile_bytes, v_head + j_cur * tile_bytes, sm); });
  raw_copies_done();
  __syncthreads();

  for (int t = 0; t < cnt; ++t) {
    const int j = j_cur;
    if (((t + 1) & 63) == 0 && t + 1 < cnt) idx_v = list_load(idx, min(t + 1 + (fresh_tid() & 63), cnt - 1));     // next 64 entries
    // The copies of tile t+1 are handed out between the MFMAs of the S^T / dP^T products of iteration t: issued
    // back to back they keep the wave at the issue stage until the texture unit has taken the last one.  They are
    // unconditional (past the end of the list the last tile is requested again, into the buffer nobody reads).
    j_cur = list_entry(min(t + 1, cnt - 1));
    set_rows(min(BKV - 1, N - 1 - j_cur * BKV));
    const char* kpn = k_head + j_cur * tile_bytes;
    const char* vpn = v_head + j_cur * tile_bytes;
    const uint32_t nx_stage = sm + ((t + 1) & 1) * STAGE_B;
    uint32_t ka = ka_off + (t & 1) * STAGE_B, kt0 = kt_off0 + (t & 1) * STAGE_B, kt1 = kt_off1 + (t & 1) * STAGE_B;
#if defined(__HIP_DEVICE_COMPILE__)
    // (keeps the XORed operand addresses out of loop-invariant hoisting: one VALU op per read instead of a dozen live
    // registers)
    asm volatile("" : "+v"(ka), "+v"(kt0), "+v"(kt1));
#endif

    // ---- S^T and dP^T - D: for each 32-key block NK MFMAs of K Q^T, then NK of V dO^T on top of -D.  LDS operands run
    // PDQ MFMAs ahead of their use; copy piece p of tile t+1 goes out after MFMA p * NM1 / NPIECE.
    constexpr int NM1 = 4 * NK, PDQ = 4, PDT = 2;
    auto frag1 = [&](int y) -> bf16x8 {
      const int kb = y / (2 * NK), rem = y % (2 * NK), kk = rem % NK;
      return lds_ld16((ka ^ (kk << 5)) + (rem < NK ? 0 : TILE_B) + kb * 32 * D * 2);
    };
    constexpr int NM2 = 4 * NMB;
    auto frag2 = [&](int y) -> bf16x8 {
      const int kb = y / (2 * NMB), cc = (y / NMB) % 2, mb = y % NMB;
      const int o = (32 * kb + 16 * cc) * D * 2;
      return join_tr(lds_tr4_at((kt0 ^ (mb << 6)) + o), lds_tr4_at((kt1 ^ (mb << 6)) + o));
    };
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    const bool tail = (j + 1) * BKV > N;
    f32x16 s[2], dp[2];
    uint32_t dsk[2][8];
    auto exp_unit = [&](auto KB, auto U) {   // P^T of two keys
      constexpr int kb = decltype(KB)::v, v = 2 * decltype(U)::v;
      s[kb][v] = fast_exp2(fmaf(s[kb][v], a.scale_log2, -lse2));
      s[kb][v + 1] = fast_exp2(fmaf(s[kb][v + 1], a.scale_log2, -lse2));
    };
    auto mask_tail = [&](auto KB) {          // keys past N (short last block): P = 0
      constexpr int kb = decltype(KB)::v;
      if (tail) {                            // (a branch: as selects it cost four instructions an element and tile)
        const int valid = N - j * BKV - kb * 32 - 4 * ((fresh_tid() & 63) >> 5);
#pragma unroll
        for (int v = 0; v < 16; ++v)
          if (8 * (v >> 2) + (v & 3) >= valid) s[kb][v] = 0.f;
      }
    };
    auto ds_unit = [&](auto KB, auto U) {    // dS^T of two keys
      constexpr int kb = decltype(KB)::v, u = decltype(U)::v;
      dsk[kb][u] = pack_bf16(s[kb][2 * u] * dp[kb][2 * u], s[kb][2 * u + 1] * dp[kb][2 * u + 1]);
    };
    bf16x8 fr[PDQ], f2[PDT];
#pragma unroll
    for (int x = 0; x < PDQ; ++x) fr[x] = frag1(x);
    static_for<0, NM1>([&](auto Y) {
      constexpr int y = decltype(Y)::v, kb = y / (2 * NK), rem = y % (2 * NK), kk = rem % NK;
      if constexpr (rem < NK) s[kb] = mfma32(fr[y % PDQ], qf[kk], kk == 0 ? zero : s[kb]);
      else                    dp[kb] = mfma32(fr[y % PDQ], dof[kk], kk == 0 ? neg_d : dp[kb]);
      if constexpr (y + PDQ < NM1) fr[y % PDQ] = frag1(y + PDQ);
      if constexpr (y % (NM1 / NPIECE) == 0) copy_piece(Int<y / (NM1 / NPIECE)>{}, kpn, vpn, nx_stage);
      if constexpr (rem >= NK) static_for<kk * 8 / NK, (kk + 1) * 8 / NK>([&](auto U) { exp_unit(Int<kb>{}, U); });
      if constexpr (rem == 2 * NK - 1) mask_tail(Int<kb>{});
      if constexpr (kb == 1 && rem < NK) static_for<kk * 8 / NK, (kk + 1) * 8 / NK>([&](auto U) { ds_unit(Int<0>{}, U); });
      if constexpr (y >= NM1 - PDT) f2[y - (NM1 - PDT)] = frag2(y - (NM1 - PDT));
      __builtin_amdgcn_sched_barrier(0);
    });
    // ---- dQ^T += K^T dS^T
    static_for<0, NM2>([&](auto Y) {
      constexpr int y = decltype(Y)::v, kb = y / (2 * NMB), cc = (y / NMB) % 2, mb = y % NMB;
      const u32x4 du = {dsk[kb][4 * cc], dsk[kb][4 * cc + 1], dsk[kb][4 * cc + 2], dsk[kb][4 * cc + 3]};
      acc[mb] = mfma32(f2[y % PDT], __builtin_bit_cast(bf16x8, du), acc[mb]);
      if constexpr (y + PDT < NM2) f2[y % PDT] = frag2(y + PDT);
      if constexpr (kb == 0) static_for<(y * 8) / (2 * NMB), ((y + 1) * 8) / (2 * NMB)>([&](auto U) { ds_unit(Int<1>{}, U); });
      __builtin_amdgcn_sched_barrier(0);
    });
    raw_copies_done();    // the copies requested in this iteration have landed
    __syncthreads();
  }

  if (parts) {                // one part of a split row; the last one to arrive adds all of them in part order
    const int64_t first = slot - part;
    const float* p0 = a.sp.pool + first * a.sp.slot_floats;
    float* ps = a.sp.pool + (first + part) * a.sp.slot_floats;
#pragma unroll
    for (int mb = 0; mb < D / 32; ++mb)
#pragma unroll
      for (int g = 0; g < 8; ++g) part_store2(ps + ((mb * 8 + g) * 256 + tid) * 2, acc[mb][2 * g], acc[mb][2 * g + 1]);
    if (!last_part(a.sp.arrive + first, parts, (int*)smem)) return;
#pragma unroll
    for (int mb = 0; mb < D / 32; ++mb)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[mb][v] = 0.f;
    for (int p = 0; p < parts; ++p) {
      const float* pp = p0 + (int64_t)p * a.sp.slot_floats;
      f32x2 x[D / 4];
#pragma unroll
      for (int c = 0; c < D / 4; ++c) x[c] = part_load2(pp + (c * 256 + tid) * 2);
#pragma unroll
      for (int c = 0; c < D / 4; ++c) {
        acc[c / 8][2 * (c % 8)] += x[c][0];
        acc[c / 8][2 * (c % 8) + 1] += x[c][1];
      }
    }
  }
  dq_store_rows<D>(a, base, i * BQ + 32 * w, lane, sm + w * (32 * D * 2), acc);
}

static hipError_t launch_dq(const void* q, const void* k, const void* v, const void* d_o, const float* lse,
                            const float* delta, const Dims& m, const int32_t* row_cnt, const int32_t* row_idx,
                            const int32_t* row_order, float scale, void* dq, const SplitPlan& plan, const SplitPlan* col_plan,
                            const int32_t* col_cnt, int32_t* col_order, hipStream_t stream) {
  DqArgs a = {};
  a.q = (const uint16_t*)q; a.k = (const uint16_t*)k; a.v = (const uint16_t*)v; a.d_o = (const uint16_t*)d_o;
  a.lse = lse; a.delta = delta; a.dq = (uint16_t*)dq;
  a.row_cnt = row_cnt; a.row_idx = row_idx; a.row_order = row_order;
  a.BH = m.B * m.H; a.H = m.H; a.N = m.N; a.Tm = m.Tm; a.Tn = m.Tn; a.chunk = (m.Tm + 7) / 8;
  a.sb = m.sb; a.sh = m.sh; a.sn = m.sn;
  a.scale = scale; a.scale_log2 = scale * LOG2E;
  a.sp = plan;
  if (plan.pool_slots && !plan.planned) {
    const hipError_t e = launch_split_plan(row_cnt, (int64_t)m.B * m.H * m.Tm, m.Tn, SPLIT_DQ, plan, stream);
    if (e != hipSuccess) return e;
  }
  if (col_plan && col_plan->pool_slots) {
    a.col_plan = plan_args(col_cnt, (int64_t)m.B * m.H * m.Tn, m.Tm, SPLIT_DKDV, *col_plan);
    a.front = 8;
  }
  if (col_plan && col_plan->stretches) {
    a.stretches = true;
    a.col_list = list_args(col_cnt, m, col_order, (int64_t)m.B * m.H * m.Tn <= 3 * col_plan->resident);
    a.orders = 8 * a.col_list.groups;
  } else if (col_plan && col_order) {
    a.col_order = order_args(col_cnt, m, col_order, 64);
    a.orders = m.B * m.H * a.col_order.groups;
  }
  const int rows = launched_rows(a.BH, a.Tm, a.chunk);
  const dim3 grid((unsigned)(a.front + plan.pool_slots + rows + a.orders)), block(256);
  if (m.d == 128) hipLaunchKernelGGL(dq_kernel<128>, grid, block, 0, stream, a);
  else            hipLaunchKernelGGL(dq_kernel<64>, grid, block, 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_bwd_dq(const void* q, const void* k, const void* v, const void* d_o, const float* lse,
                         const float* delta, const Dims& m, const int32_t* row_cnt, const int32_t* row_idx,
                         const int32_t* row_order, float scale, void* dq, const SplitPlan& plan, hipStream_t stream) {
  return launch_dq(q, k, v, d_o, lse, delta, m, row_cnt, row_idx, row_order, scale, dq, plan, nullptr, nullptr, nullptr, stream);
}

hipError_t launch_bwd_dq_columns(const void* q, const void* k, const void* v, const void* d_o, const float* lse,
                                 const float* delta, const Dims& m, const int32_t* row_cnt, const int32_t* row_idx,
                                 const int32_t* row_order, float scale, void* dq, const SplitPlan& plan,
                                 const int32_t* col_cnt, int32_t* col_order, const SplitPlan& col_plan, hipStream_t stream) {
  return launch_dq(q, k, v, d_o, lse, delta, m, row_cnt, row_idx, row_order, scale, dq, plan, &col_plan, col_cnt, col_order,
                   stream);
}

}  // namespace spa2
