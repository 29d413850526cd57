// Block-sparse attention forward (Alg. 1 steps 7-21; Sec. 2.1) for gfx950.
//
// One workgroup (4 waves) per query block of 128 rows; wave w owns rows
// 32w..32w+31.  The workgroup walks the selected key blocks of its row of the
// block mask; each K/V tile (64 x d) is staged through LDS once and shared by
// the four waves.
//
// Everything is computed transposed so that a lane owns ONE query row:
//   S^T (keys x queries) = K_j Q_i^T      A = K rows from LDS, B = Q^T held in registers
//   O^T (d x queries)   += V_j^T P^T      A = V^T via transposing LDS reads, B = P^T
// The accumulator layout of S^T (lane = query, registers = keys) is exactly the
// B-operand layout the second product wants, so P never leaves registers, and
// the running maximum / sum of Alg. 1 (m_ij, l_ij) are per-lane scalars that
// need one exchange between the two halves of the wave per tile.
#include "row_map.h"
#include "spa2_device.h"
#include "spa2_internal.h"

namespace spa2 {

struct FwdArgs {
  const uint16_t* q; const uint16_t* k; const uint16_t* v;
  uint16_t* o; uint16_t* o_res; float* lse;
  const int32_t* row_cnt; const int32_t* row_idx; const int32_t* row_order;
  int BH, H, N, Tm, Tn, chunk;
  int64_t sb, sh, sn;
  float scale_log2;     // scale * log2(e): softmax is evaluated with exp2
  SplitPlan sp;         // long rows cut into parts (split.hip); sp.pool_slots == 0: every row is walked whole
};

// Partial result of one part of a split row: the unnormalised accumulator as [pair of accumulator registers][thread],
// so that the 64 lanes of a wave write and read consecutive 8-byte pieces, then per thread the running maximum (log2
// units) and the row sum, both already combined over the two halves of the wave.
template <int D> constexpr int fwd_slot_floats() { return 256 * (D / 2) + 512; }
size_t fwd_slot_bytes(const Dims& m) { return (size_t)(m.d == 128 ? fwd_slot_floats<128>() : fwd_slot_floats<64>()) * 4; }

// O_i = diag(l)^-1 O (Alg. 1 step 18) -> bf16 (+ optional residual), LSE = m ln 2 + log l.  q0: first row of the wave;
// area: LDS of the wave's own for both outputs, which the other waves may still be reading.
template <int D>
__device__ __forceinline__ void fwd_store_rows(const FwdArgs& a, int bh, int64_t base, int q0, int lane, uint32_t area,
                                               const f32x16 (&oacc)[D / 32], float m_run, float l_tot) {
  const float inv = 1.f / l_tot;
  const int r32 = lane & 31, hf = lane >> 5, valid = min(32, a.N - q0);
  constexpr int RES = 32 * D * 2;
  __syncthreads();
#pragma unroll
  for (int mb = 0; mb < D / 32; ++mb)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      float x[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = oacc[mb][4 * g + e] * inv;
      const u32x2 pk2 = {pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3])};
      row_piece_put<D>(area, r32, 4 * mb + g, hf, pk2);
      if (a.o_res) {      // what the rounding to bf16 dropped, itself rounded to bf16
        const float r0 = x[0] - __builtin_bit_cast(float, pk2[0] << 16);
        const float r1 = x[1] - __builtin_bit_cast(float, pk2[0] & 0xffff0000u);
        const float r2 = x[2] - __builtin_bit_cast(float, pk2[1] << 16);
        const float r3 = x[3] - __builtin_bit_cast(float, pk2[1] & 0xffff0000u);
        const u32x2 pr = {pack_bf16(r0, r1), pack_bf16(r2, r3)};
        row_piece_put<D>(area + RES, r32, 4 * mb + g, hf, pr);
      }
    }
  const int64_t off = base + (int64_t)q0 * a.sn;
  rows_store<D>(area, a.o + off, a.sn, valid, lane);
  if (a.o_res) rows_store<D>(area + RES, a.o_res + off, a.sn, valid, lane);
  if (hf == 0 && r32 < valid) a.lse[(int64_t)bh * a.N + q0 + r32] = m_run * LN2 + __logf(l_tot);
}

template <int D>
__global__ __launch_bounds__(256, 2) void fwd_kernel(FwdArgs a) {
  constexpr int NK = D / 16, NMB = D / 32;           // contraction steps of S, output blocks of O
  // Three K and two V tiles, XOR-swizzled and unpadded (the layout a direct global -> LDS copy can write); two
  // workgroups of 80 KB share a compute unit.  (Aligned: compile-time parts are XORed into addresses.)
  constexpr int TILE_B = BKV * D * 2, V_SLOTS = 3 * TILE_B;
  __shared__ __align__(1024) unsigned char smem[5 * TILE_B];

  // Which row, and which part of its list.  The first sp.pool_slots workgroups of the launch are the parts of split
  // rows; the others take one row each, unless it is split.
  int bh, i, part = 0, parts = 0, part_len = 0;
  bool whole = false;         // a row of the plan that may be split: its parts are the first workgroups
  int slot = blockIdx.x;
  if (a.sp.fixed_len) {       // a small launch: the sizes say which part of which row (with_fixed_parts)
    const int rows = stretch_wgs(a.BH * a.Tm);
    const HeadBlock hb = stretch_row(blockIdx.x % rows, a.BH, a.Tm);
    if (!hb.valid) return;
    bh = hb.bh; i = hb.blk;
    const int unit = bh * a.Tm + i, all = min(max(a.row_cnt[unit], 0), a.Tn);
    part = blockIdx.x / rows;
    parts = all > a.sp.fixed_len ? (all + a.sp.fixed_len - 1) / a.sp.fixed_len : 0;
    if (part >= max(parts, 1)) return;
    if (parts) part_len = (all + parts - 1) / parts;
    slot = unit * a.sp.fixed_parts + part;
  } else if ((int)blockIdx.x < a.sp.pool_slots) {
    if ((int)blockIdx.x >= scalar_ld(a.sp.header)) return;
    const int32_t* pt = a.sp.part_table + 4 * blockIdx.x;
    const int unit = scalar_ld(pt);
    part = scalar_ld(pt + 1); parts = scalar_ld(pt + 2); part_len = scalar_ld(pt + 3);
    bh = unit / a.Tm; i = unit % a.Tm;
  } else {
    const int wg = blockIdx.x - a.sp.pool_slots;
    const HeadBlock hb = launched_row(a.sp, wg, a.BH, a.Tm, a.chunk);
    if (!hb.valid) return;
    bh = hb.bh;
    // optional launch order: position hb.blk of this head's schedule -> query block (clamped: caller data)
    i = a.row_order ? min(max(a.row_order[(int64_t)bh * a.Tm + hb.blk], 0), a.Tm - 1) : hb.blk;
    whole = a.sp.pool_slots != 0;
  }
  const int64_t base = (int64_t)(bh / a.H) * a.sb + (int64_t)(bh % a.H) * a.sh;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);     // wave-uniform, in a scalar register
  const int r32 = lane & 31, hf = lane >> 5;
  const int N = a.N;
  // counts and indices come from the caller's pattern: clamp them so that a corrupt list cannot
  // address memory outside the tensors
  const int64_t unit = (int64_t)bh * a.Tm + i;
  int cnt = min(max(a.row_cnt[unit], 0), a.Tn);
  const int split_at = *(whole ? a.sp.unit_slot + unit : a.row_cnt + unit);
  const int first = part * part_len;         // entries [first, first + part_len) of the list of a split row (never empty)
  const int32_t* idx = a.row_idx + unit * a.Tn + first;
  // The list's first 64 entries and the queries are requested before the count (or whether the row is split) is known:
  // one wait for all of these instead of three, each a round trip to memory.  (Measured, us, before / after: 1000 tokens,
  // 2 heads 14.8 / 14.3, 4 samples of 1281 tokens 32.5 / 31.9, 20,010 tokens, 6 heads, d = 64 64.0 / 63.6; the same in dQ 31.0 /
  // 30.4 and 72.1 / 71.4.  In dK/dV it gave 0.3 us on the short ones and cost 2.6 of 126 on the last, so it is not there.)
  int idx_v = idx[min(lane, a.Tn - 1 - first)];
  const int qrow = i * BQ + w * 32 + r32;
  // Q^T fragments (B operand): lane = query row, 8 consecutive channels per 16-wide k step.
  const int qrow_ld = qrow < N ? qrow : N - 1;
  bf16x8 qf[D / 16];
  {
    const uint16_t* qp = a.q + base + (int64_t)qrow_ld * a.sn + 8 * hf;
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) qf[kk] = *(const bf16x8*)(qp + 16 * kk);
  }
  requested();
  if (whole && split_at >= 0) return;
  if (parts) cnt = min(cnt - first, part_len);

  if (cnt == 0) {   // a row without any selected block (never produced by the masker): O = 0, LSE = -inf
    if (qrow < N) {
      uint16_t* op = a.o + base + (int64_t)qrow * a.sn + (D / 2) * hf;
#pragma unroll
      for (int c = 0; c < D / 16; ++c) *(u32x4*)(op + 8 * c) = u32x4{0, 0, 0, 0};
      if (a.o_res) {
        uint16_t* rp = a.o_res + (op - a.o);
#pragma unroll
        for (int c = 0; c < D / 16; ++c) *(u32x4*)(rp + 8 * c) = u32x4{0, 0, 0, 0};
      }
      if (hf == 0) a.lse[(int64_t)bh * N + qrow] = -INFINITY;
    }
    return;
  }

  // K/V tiles are copied global -> LDS directly.  The destination of a wave-wide 16-byte-per-lane copy is linear (wave
  // base + 16 * lane), so the swizzle is applied on the source side: the lane that fills chunk position pc of a row
  // fetches logical chunk pc ^ swz(row).  Thread t fills chunk position t % CPR of rows t / CPR + r * RSTEP; RSTEP is a
  // multiple of 16 rows, so the swizzle term is the same for every r.  Rows past N (short last block) are clamped to the
  // last token: their keys are masked out of the softmax and their P is exactly zero.  The lane offsets are computed
  // again only when the number of valid rows changes.
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
  auto set_rows = [&](int j) {               // for the tile of key block j (uniform)
    const int last = min(BKV - 1, N - 1 - j * BKV);
    if (last == rows_set) return;
    rows_set = last;
    const int t = fresh_tid(), ld_row = t / CPR, ld_c8 = ((t % CPR) ^ swz<D>(ld_row)) * 8;
#pragma unroll
    for (int r = 0; r < CH; ++r) voff[r] = (uint32_t)((min(ld_row + RSTEP * r, last) * a.sn + ld_c8) * 2);
  };
  const uint32_t sm = lds_addr_of(smem), sm_w = sm + w * 1024;
  const char* k_head = (const char*)(a.k + base);
  const char* v_head = (const char*)(a.v + base);
  const uint64_t tile_bytes = (uint64_t)a.sn * (2 * BKV);
  auto copy_tile = [&](const char* src, uint32_t slot) {
    static_for<0, CH>([&](auto R) { raw_copy16_to_lds_at<decltype(R)::v * 4096>(src, voff[decltype(R)::v], sm_w + slot); });
  };

  f32x16 oacc[NMB];
#pragma unroll
  for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
    for (int v = 0; v < 16; ++v) oacc[mb][v] = 0.f;
  float m_run = -INFINITY;   // running maximum, in log2 units (already multiplied by scale_log2)
  float l_run = 0.f;         // running sum over THIS lane's keys; the two halves are added at the end

  // per-lane LDS byte offsets inside a tile.  K row reads: row 32kb + r32, logical chunk 2kk + hf; the part of the chunk
  // index that depends on kk is XORed in as (kk << 5).  V transposing reads: rows (16-row group) + 8*which + 4hf +
  // (s16>>2), columns 32mb + 16hb + 4(s16&3); the part that depends on mb is XORed in as (mb << 6).
  const int s16 = lane & 15, hb16 = (lane >> 4) & 1;
  const uint32_t k_off = sm + 2 * swz_idx<D>(r32, 8 * hf);
  const uint32_t v_off0 = sm + V_SLOTS + 2 * swz_idx<D>(4 * hf + (s16 >> 2), 16 * hb16 + 4 * (s16 & 3));
  const uint32_t v_off1 = sm + V_SLOTS + 2 * swz_idx<D>(8 + 4 * hf + (s16 >> 2), 16 * hb16 + 4 * (s16 & 3));

  // The list of selected key blocks, 64 entries at a time in one register (lane l holds entry 64c + l): reading an entry
  // is a lane read, not a memory access whose result the loop would have to wait for.
  // Where in its list a row starts is a free choice (the online softmax does not depend on the order of the
  // tiles, up to rounding), and it is used to keep the rows that run on one XCD at the same time close
  // together in key space: query block i starts at the first selected block at or after (i mod 64) / 64 of
  // the key range and wraps around.  An XCD takes consecutive query blocks, and its workgroups start as slots
  // free up, one row-duration spread over its 64 slots; so a row that starts 1/64 of a row-duration later
  // also starts 1/64 of the key range further on: all of them sweep the keys together and share K/V tiles
  // through the XCD's L2.  The start depends on the row alone, so results do not depend on the launch order.
  int pos = 0;                               // place in the list of the next entry (idx_v: the 64 entries around it)
  {
    const int start_blk = (int)(((int64_t)(i & 63) * a.Tn) >> 6);
    pos = __builtin_popcountll(__builtin_amdgcn_ballot_w64(lane < cnt && idx_v < start_blk));
    for (int c = 64; c < cnt; c += 64) {
      idx_v = idx[min(c + lane, cnt - 1)];
      pos += __builtin_popcountll(__builtin_amdgcn_ballot_w64(c + lane < cnt && idx_v < start_blk));
    }
    pos = __builtin_amdgcn_readfirstlane(pos);
    if (pos >= cnt) pos = 0;
    if (cnt > 64) idx_v = list_load(idx, min((pos & ~63) + lane, cnt - 1));
  }
  int left = cnt - 1;                        // entries behind the one at pos (past the end the last one is taken again)
  auto next_entry = [&]() -> int {
    const int j = min(max(__builtin_amdgcn_readlane(idx_v, pos & 63), 0), a.Tn - 1);
    if (left > 0) {
      --left;
      pos = pos + 1 == cnt ? 0 : pos + 1;
      if (cnt > 64 && (pos & 63) == 0) idx_v = list_load(idx, min(pos + (fresh_tid() & 63), cnt - 1));
    }
    return j;
  };

  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  constexpr int PD = 4, PDV = 4;             // how many MFMAs ahead an LDS operand is requested
  uint32_t pk[2][8];
  // P^T = exp(S^T - m) (step 12) of two keys, rounded to bf16 for the second product; the row sum (step 13) is taken
  // over the rounded values, so numerator and denominator use the same weights
  auto exp_unit = [&](const f32x16 (&s)[2], auto U) {
    constexpr int kb = decltype(U)::v / 8, u = decltype(U)::v % 8;
    const float p0 = fast_exp2(fmaf(s[kb][2 * u], a.scale_log2, -m_run));
    const float p1 = fast_exp2(fmaf(s[kb][2 * u + 1], a.scale_log2, -m_run));
    pk[kb][u] = pack_bf16(p0, p1);
    l_run = dot2_ones(pk[kb][u], l_run);
  };
  // keys past N (short last block) do not take part in the softmax
  auto mask_tail = [&](f32x16 (&s)[2], int j) {
    if ((j + 1) * BKV > N) {
      const int valid = N - j * BKV - 4 * ((fresh_tid() & 63) >> 5);
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int v = 0; v < 16; ++v)
          if (kb * 32 + 8 * (v >> 2) + (v & 3) >= valid) s[kb][v] = -INFINITY;
    }
  };
  // running maximum (Alg. 1 step 11); the accumulators are rescaled (steps 13-14) only when some row's maximum moved:
  // after the first few tiles it rarely does, and the branch is uniform over the wave
  auto new_max = [&](float mx) {
    mx = max_halves(mx);
    const float m_new = fmaxf(m_run, mx * a.scale_log2);
    if (__builtin_amdgcn_ballot_w64(m_new != m_run) != 0) {
      const float alpha = fast_exp2(m_run - m_new);
      l_run *= alpha;
#pragma unroll
      for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
        for (int v = 0; v < 16; ++v) oacc[mb][v] *= alpha;
      m_run = m_new;
    }
  };
  auto k_frag = [&](uint32_t ka, int y) -> bf16x8 {            // y = kb * NK + kk
    return lds_ld16((ka ^ ((y % NK) << 5)) + (y / NK) * 32 * D * 2);
  };
  auto v_frag = [&](uint32_t v0, uint32_t v1, int x) -> bf16x8 {       // x = (kb, cc, mb)
    const int o = (x / NMB) * 16 * D * 2, mb = x % NMB;
    return join_tr(lds_tr4_at((v0 ^ (mb << 6)) + o), lds_tr4_at((v1 ^ (mb << 6)) + o));
  };
  auto p_frag = [&](int x) -> bf16x8 {       // P^T of the 16 keys (kb, cc)
    const int kb = x / (2 * NMB), cc = (x / NMB) % 2;
    return __builtin_bit_cast(bf16x8, u32x4{pk[kb][4 * cc], pk[kb][4 * cc + 1], pk[kb][4 * cc + 2], pk[kb][4 * cc + 3]});
  };

  // Bound: the board's power (1.70 GHz).  Pipeline: iteration t computes S of tile t+1 with the exponentials of tile t between the products, then adds
  // V P of tile t with the rest of them and the maximum of tile t+1 between: a wave's vector arithmetic runs behind its
  // own products.  Meanwhile V of tile t+1 (whose slot tile t-1 has left) and K of tile t+3 (slot of tile t) are on
  // their way; all but the latter have landed at the barrier that ends the iteration.  The copies are handed out between
  // the products: issued back to back they would keep the wave at the issue stage until the texture unit has taken the
  // last one.  They are unconditional (past the end of the list its last tile is requested again).
  // Measured against S, softmax and V P one after the other with tiles staged through registers, us, before / after
  // (same bits): 75,600 tokens, 40 heads at 94 % / 97 % sparsity 8042 / 7800 and 4235 / 4085; 32,760 tokens, 12 heads
  // 904 / 870, 3 heads and every tile 1661 / 1604; 3500 instead of 3700 cycles a tile and wave at two waves per SIMD.
  uint32_t ks0 = 0, ks1 = TILE_B, ks2 = 2 * TILE_B;            // slots of K of tiles t, t+1, t+2
  int j1, j2, j3;                                              // key blocks of tiles t+1, t+2, t+3
  f32x16 sA[2], sB[2];
  {
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) asm volatile("" : "+v"(qf[kk]));   // (Q is waited for before the copies, not with them)
#endif
    const int j0 = next_entry();
    j1 = next_entry(); j2 = next_entry();
    set_rows(j0);
    copy_tile(k_head + j0 * tile_bytes, ks0);
    copy_tile(v_head + j0 * tile_bytes, V_SLOTS);
    set_rows(j1);
    copy_tile(k_head + j1 * tile_bytes, ks1);
    set_rows(j2);
    copy_tile(k_head + j2 * tile_bytes, ks2);
    j3 = next_entry();
    raw_copies_left<3 * CH>();
    __syncthreads();
    bf16x8 fr[PD];
#pragma unroll
    for (int x = 0; x < PD; ++x) fr[x] = k_frag(k_off, x);
    static_for<0, 2 * NK>([&](auto Y) {
      constexpr int y = decltype(Y)::v, kb = y / NK, kk = y % NK;
      sA[kb] = mfma32(fr[y % PD], qf[kk], kk == 0 ? zero : sA[kb]);
      if constexpr (y + PD < 2 * NK) fr[y % PD] = k_frag(k_off, y + PD);
      __builtin_amdgcn_sched_barrier(0);
    });
    mask_tail(sA, j0);
    float mx = sA[0][0];
#pragma unroll
    for (int v = 1; v < 32; ++v) mx = fmaxf(mx, sA[v / 16][v % 16]);
    m_run = max_halves(mx) * a.scale_log2;
    raw_copies_left<CH>();
    __syncthreads();
  }
  auto step = [&](const f32x16 (&sc)[2], f32x16 (&sn)[2], int t) {     // sc: S of tile t, sn: of tile t+1
    constexpr int E1 = D == 128 ? 10 : 8;    // exponential units (of 16) that run between the S products
    uint32_t ka = k_off + ks1, v0 = v_off0 + (t & 1) * TILE_B, v1 = v_off1 + (t & 1) * TILE_B;
#if defined(__HIP_DEVICE_COMPILE__)
    // (keeps the XORed operand addresses out of loop-invariant hoisting: one VALU op per read instead of a dozen live
    // registers)
    asm volatile("" : "+v"(ka), "+v"(v0), "+v"(v1));
#endif
    const char* vpn = v_head + j1 * tile_bytes;
    const char* kpn = k_head + j3 * tile_bytes;
    const uint32_t v_dst = sm_w + V_SLOTS + ((t + 1) & 1) * TILE_B, k_dst = sm_w + ks0;
    bf16x8 fr[PD], vf[PDV];
#pragma unroll
    for (int x = 0; x < PD; ++x) fr[x] = k_frag(ka, x);
    set_rows(j1);
    // S^T = K_j Q_i^T of tile t+1: two 32-key blocks
    static_for<0, 2 * NK>([&](auto Y) {
      constexpr int y = decltype(Y)::v, kb = y / NK, kk = y % NK, piece = y / 2;
      sn[kb] = mfma32(fr[y % PD], qf[kk], kk == 0 ? zero : sn[kb]);
      if constexpr (y + PD < 2 * NK) fr[y % PD] = k_frag(ka, y + PD);
      if constexpr (y == 2 * CH) set_rows(j3);
      if constexpr (y % 2 == 0) {
        if constexpr (piece < CH) raw_copy16_to_lds_at<piece * 4096>(vpn, voff[piece], v_dst);
        else                      raw_copy16_to_lds_at<(piece - CH) * 4096>(kpn, voff[piece - CH], k_dst);
      }
      static_for<y * E1 / (2 * NK), (y + 1) * E1 / (2 * NK)>([&](auto U) { exp_unit(sc, U); });
      if constexpr (y >= 2 * NK - PDV) vf[y - (2 * NK - PDV)] = v_frag(v0, v1, y - (2 * NK - PDV));
      __builtin_amdgcn_sched_barrier(0);
    });
    mask_tail(sn, j1);
    // O^T += V^T P^T of tile t (step 14).  MFMA x uses key slots 32kb + 16cc + 4hf + {0..3} and + 8 (the order the
    // accumulator of S^T holds them in) of output block mb.
    float mx = -INFINITY;
    static_for<0, 4 * NMB>([&](auto X) {
      constexpr int x = decltype(X)::v, mb = x % NMB, H = 2 * NMB;
      oacc[mb] = mfma32(vf[x % PDV], p_frag(x), oacc[mb]);
      if constexpr (x + PDV < 4 * NMB) vf[x % PDV] = v_frag(v0, v1, x + PDV);
      if constexpr (x < H) {
        static_for<E1 + x * (16 - E1) / H, E1 + (x + 1) * (16 - E1) / H>([&](auto U) { exp_unit(sc, U); });
      } else {
        static_for<(x - H) * 32 / H, (x - H + 1) * 32 / H>([&](auto V) { mx = fmaxf(mx, sn[decltype(V)::v / 16][decltype(V)::v % 16]); });
      }
      __builtin_amdgcn_sched_barrier(0);
    });
    raw_copies_left<CH>();
    __syncthreads();
    new_max(mx);
    const uint32_t k = ks0; ks0 = ks1; ks1 = ks2; ks2 = k;
    j1 = j2; j2 = j3; j3 = next_entry();
  };
  auto last_step = [&](const f32x16 (&sc)[2], int t) {         // V P of the last tile
    const uint32_t v0 = v_off0 + (t & 1) * TILE_B, v1 = v_off1 + (t & 1) * TILE_B;
    bf16x8 vf[PDV];
#pragma unroll
    for (int x = 0; x < PDV; ++x) vf[x] = v_frag(v0, v1, x);
    static_for<0, 8>([&](auto U) { exp_unit(sc, U); });
    static_for<0, 4 * NMB>([&](auto X) {
      constexpr int x = decltype(X)::v, mb = x % NMB, H = 2 * NMB;
      oacc[mb] = mfma32(vf[x % PDV], p_frag(x), oacc[mb]);
      if constexpr (x + PDV < 4 * NMB) vf[x % PDV] = v_frag(v0, v1, x + PDV);
      if constexpr (x < H) static_for<8 + x * 8 / H, 8 + (x + 1) * 8 / H>([&](auto U) { exp_unit(sc, U); });
      __builtin_amdgcn_sched_barrier(0);
    });
    raw_copies_done();       // (nothing may land in the LDS once this workgroup is through with it)
  };
  int t = 0;
  for (; t + 2 < cnt; t += 2) {
    step(sA, sB, t);
    step(sB, sA, t + 1);
  }
  if (t + 1 < cnt) {
    step(sA, sB, t);
    ++t;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) sA[kb] = sB[kb];
  }
  last_step(sA, t);

  const float l_tot = sum_halves(l_run);
  constexpr int OUT_B = 2 * 32 * D * 2;      // a wave's rows of O and of the residual, on their way out
  static_assert(4 * OUT_B <= 5 * TILE_B, "the outputs of four waves fit the tiles' LDS");
  if (parts) {                // one part of a split row
    const int64_t first = slot - part;
    float* ps = a.sp.pool + (first + part) * a.sp.slot_floats;
#pragma unroll
    for (int mb = 0; mb < D / 32; ++mb)
#pragma unroll
      for (int g = 0; g < 8; ++g) part_store2(ps + ((mb * 8 + g) * 256 + tid) * 2, oacc[mb][2 * g], oacc[mb][2 * g + 1]);
    part_store2(ps + 256 * (D / 2) + 2 * tid, m_run, l_tot);
    if (!last_part(a.sp.arrive + first, parts, (int*)smem)) return;
    // The last part to arrive combines all of them, in part order (so the result does not depend on which one that
    // is): m = max m_p, l = sum l_p 2^(m_p - m), O = sum O_p 2^(m_p - m) / l.
    const float* p0 = a.sp.pool + first * a.sp.slot_floats;
    float m = -INFINITY, l = 0.f;
    for (int p = 0; p < parts; p += 4) {       // four loads in flight per step
      float mp[4];
#pragma unroll
      for (int x = 0; x < 4; ++x) mp[x] = part_load2(p0 + (int64_t)min(p + x, parts - 1) * a.sp.slot_floats + 256 * (D / 2) + 2 * tid)[0];
      m = fmaxf(fmaxf(m, fmaxf(mp[0], mp[1])), fmaxf(mp[2], mp[3]));
    }
#pragma unroll
    for (int mb = 0; mb < D / 32; ++mb)
#pragma unroll
      for (int v = 0; v < 16; ++v) oacc[mb][v] = 0.f;
    for (int p = 0; p < parts; ++p) {
      const float* pp = p0 + (int64_t)p * a.sp.slot_floats;
      f32x2 x[D / 4];
#pragma unroll
      for (int c = 0; c < D / 4; ++c) x[c] = part_load2(pp + (c * 256 + tid) * 2);
      const f32x2 ml = part_load2(pp + 256 * (D / 2) + 2 * tid);
      const float sc = fast_exp2(ml[0] - m);
      l = fmaf(ml[1], sc, l);
#pragma unroll
      for (int c = 0; c < D / 4; ++c) {
        oacc[c / 8][2 * (c % 8)] = fmaf(x[c][0], sc, oacc[c / 8][2 * (c % 8)]);
        oacc[c / 8][2 * (c % 8) + 1] = fmaf(x[c][1], sc, oacc[c / 8][2 * (c % 8) + 1]);
      }
    }
    fwd_store_rows<D>(a, bh, base, i * BQ + 32 * w, lane, sm + w * OUT_B, oacc, m, l);
    return;
  }
  // O_i = diag(l)^-1 O (step 18) and the log-sum-exp the backward pass needs
  fwd_store_rows<D>(a, bh, base, i * BQ + 32 * w, lane, sm + w * OUT_B, oacc, m_run, l_tot);
}

hipError_t launch_fwd(const void* q, const void* k, const void* v, const Dims& m, const int32_t* row_cnt,
                      const int32_t* row_idx, const int32_t* row_order, float scale, void* o, void* o_res,
                      float* lse, const SplitPlan& plan, hipStream_t stream) {
  FwdArgs a;
  a.q = (const uint16_t*)q; a.k = (const uint16_t*)k; a.v = (const uint16_t*)v;
  a.o = (uint16_t*)o; a.o_res = (uint16_t*)o_res; a.lse = lse;
  a.row_cnt = row_cnt; a.row_idx = row_idx; a.row_order = row_order;
  a.BH = m.B * m.H; a.H = m.H; a.N = m.N; a.Tm = m.Tm; a.Tn = m.Tn;
  a.chunk = (m.Tm + 7) / 8;
  a.sb = m.sb; a.sh = m.sh; a.sn = m.sn;
  a.scale_log2 = scale * LOG2E;
  a.sp = plan;
  if (plan.pool_slots && !plan.planned) {
    const hipError_t e = launch_split_plan(row_cnt, (int64_t)m.B * m.H * m.Tm, m.Tn, SPLIT_FWD, plan, stream);
    if (e != hipSuccess) return e;
  }
  const dim3 grid((unsigned)(plan.fixed_len ? plan.fixed_parts * stretch_wgs(a.BH * a.Tm)
                                            : plan.pool_slots + launched_rows(a.BH, a.Tm, a.chunk))), block(256);
  if (m.d == 128) hipLaunchKernelGGL(fwd_kernel<128>, grid, block, 0, stream, a);
  else            hipLaunchKernelGGL(fwd_kernel<64>, grid, block, 0, stream, a);
  return hipGetLastError();
}

}  // namespace spa2
