// Block-sparse attention backward, key-block side: dK and dV (see bwd.hip for the formulas and the other two
// kernels).  This file is compiled with -mllvm -amdgpu-mfma-vgpr-form: the S / dP products then leave their
// results in ordinary vector registers, where the exp / dS arithmetic reads them directly, while the dK / dV
// accumulators are pinned to the accumulation registers through mfma32_acc below.
#include "spa2_device.h"
#include "spa2_internal.h"
#include "work_queue.h"

namespace spa2 {

// C += A B with C held in accumulation registers (the compiler allocates them there and never moves them).
// The compiler does not know that this is a matrix instruction and adds no wait states around it, so they are
// written here: an operand register that a vector ALU instruction has just written must not be read by the very
// next instruction (measured: one wait state is enough; two are kept).
__device__ __forceinline__ void mfma32_acc(bf16x8 a, bf16x8 b, f32x16& c) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
#endif
}

// ------------------------------------------------------------------ dK, dV
struct DkvArgs {
  const uint16_t* q; const uint16_t* k; const uint16_t* v; const uint16_t* d_o;
  const float* lse; const float* delta; uint16_t* dk; uint16_t* dv;
  const int32_t* col_cnt; const int32_t* col_idx; const int32_t* col_order;
  int BH, H, N, Tm, Tn, chunk;
  int64_t sb, sh, sn;
  float scale, scale_log2;
  SplitPlan sp;         // long columns cut into parts (split.hip); sp.pool_slots == 0: every column is walked whole
};

// Partial result of one part of a split column: the fp32 sums of the two waves, dK^T then dV^T, in the order
// [tensor][finishing wave][output block][pair of registers][lane][register in the pair].
template <int D> constexpr int dkdv_slot_floats() { return 2 * 2 * (D / 32) * 16 * 64; }
size_t dkdv_slot_bytes(const Dims& m) { return (size_t)(m.d == 128 ? dkdv_slot_floats<128>() : dkdv_slot_floats<64>()) * 4; }

// The last part of a split column to arrive adds all of them in part order and stores the rows that wave w finishes, key0w ..
// (area: 32 * D * 2 bytes of LDS of the wave's own).
template <int D>
__device__ __forceinline__ void dkdv_merge(const DkvArgs& a, const WorkItem& item, int64_t base, int key0w, int w, int lane,
                                           uint32_t area) {
  constexpr int NMB = D / 32;
  const float* p0 = a.sp.pool + (int64_t)(item.slot - item.part) * a.sp.slot_floats + 2 * lane;
#pragma unroll
  for (int round = 0; round < 2; ++round) {
    f32x2 x[NMB * 8];
#pragma unroll
    for (int c = 0; c < NMB * 8; ++c) x[c] = f32x2{0.f, 0.f};
    for (int p = 0; p < item.parts; ++p) {
      const float* ps = p0 + (int64_t)p * a.sp.slot_floats + (round * 2 + w) * NMB * 8 * 128;
      f32x2 y[NMB * 8];
#pragma unroll
      for (int c = 0; c < NMB * 8; ++c) y[c] = part_load2(ps + c * 128);
#pragma unroll
      for (int c = 0; c < NMB * 8; ++c) { x[c][0] += y[c][0]; x[c][1] += y[c][1]; }
    }
    const float sc = round == 0 ? -a.scale : 1.f;
#pragma unroll
    for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x2 lo = x[mb * 8 + 2 * g], hi = x[mb * 8 + 2 * g + 1];
        u32x2 pk2 = {pack_bf16(lo[0] * sc, lo[1] * sc), pack_bf16(hi[0] * sc, hi[1] * sc)};
        row_piece_put<D>(area, lane & 31, 4 * mb + g, lane >> 5, pk2);
      }
    rows_store<D>(area, (round == 0 ? a.dk : a.dv) + base + (int64_t)key0w * a.sn, a.sn, a.N - key0w, lane);
  }
}

// Head dimension 128: one workgroup of two waves per key block j (64 keys); one wave per SIMD (512 registers), four per CU.
// The query blocks that selected j are taken in halves of 64 rows; wave w owns the 32 queries 32w.. of the half
// and ALL 64 keys of the block.  It keeps K_j^T, V_j^T (B operands) and its dK^T, dV^T accumulators (d x 64
// keys each) in registers for the whole column, so every operand fragment that comes from LDS feeds two MFMAs
// (one per 32-key half), and a wave only ever reads its own 32 rows of Q and dO:
//   S  (q x keys) = Q_i K_j^T        A = Q rows from LDS,  B = K^T fragments (registers)
//   dP (q x keys) = dO_i V_j^T       A = dO rows from LDS, B = V^T fragments (registers)
//   P = exp(S - LSE), dS = P * (dP - D)      accumulator layout: lane = key, registers = queries
//   dV^T (d x keys) += dO_i^T P      A = dO^T through transposing LDS reads, B = P  (registers)
//   dK^T (d x keys) += Q_i^T dS      A = Q^T  through transposing LDS reads, B = dS (registers)
// Because no wave reads another wave's rows, each wave stages its own rows (global -> LDS directly, XOR-swizzled,
// double-buffered) and waits only for its own copies: there is no workgroup barrier in the loop.  Q rows, LSE and D of
// the next step are requested between the S products and dO rows between the dP products, so every copy has a whole
// step to land and the texture unit is not asked for sixteen of them at once.
// With a single wave per SIMD the vector arithmetic has to hide behind that wave's own MFMAs.  The order of a step is
//   16 S products          | copies; D is read from LDS into the accumulators of dP
//   16 dP products         | exp(S - LSE) of the first 20 of the 32 values of a lane
//   16 dV products         | the other exponentials (first half), dS of the first 16 queries (second half)
//   16 dK products         | dS of the other 16 queries, first row fragments of the next step
// (counts for d = 128).  dV comes before dK because it needs P alone: dS is never waited for.  dP starts from D and
// V^T is held negated, so that the products give D - dP and dS costs one multiplication an element.
// Bound: the board's power, then issue slots: 3480 cycles a step for 2048 of matrix products (4170 before this order,
// when dS of the first 16 queries had no product to hide behind, LSE and D were waited for as they were read and every
// copy stood behind a branch), 1.80 instead of 1.95 GHz.  Measured, us, before / after: 75,600 tokens, 40 heads
// 14772 / 13440; 32,760 tokens, 12 heads 1026 / 921.
// The two waves add their partial sums through LDS at the end of the column.
template <int D>
__device__ __forceinline__ void dkdv_item(const DkvArgs& a, const WorkItem& item, Walk& walk, unsigned char* smem,
                                          unsigned char* stat_s) {
  constexpr int QW = 32;                             // query rows per wave and step
  constexpr int HQ = 64;                             // query rows per workgroup and step
  constexpr int NK = D / 16;                         // 16-wide contraction steps over the head dimension
  constexpr int NMB = D / 32;                        // 32-channel output blocks
  constexpr int CPR = D / 8;                         // 16-byte chunks per row
  constexpr int RPI = 64 / CPR;                      // rows that one wave-wide copy instruction covers
  constexpr int NCP = QW / RPI;                      // copy instructions per tensor and step
  constexpr int TILE_B = QW * D * 2;                 // bytes of one wave's 32-row tile
  constexpr int STAGE_B = 2 * TILE_B;                // Q rows, then dO rows
  constexpr int STAT_B = 512;                        // LSE of the 32 rows at +0, D at +256
  const int bh = item.bh, j = item.blk, part = item.part, parts = item.parts, part_len = item.part_len;
  const int64_t base = (int64_t)(bh / a.H) * a.sb + (int64_t)(bh % a.H) * a.sh;
  const int lane = fresh_lane(), w = walk.wave;
  const int r32 = lane & 31, hf = lane >> 5;
  const int N = a.N;
  int cnt = min(max(a.col_cnt[(int64_t)bh * a.Tn + j], 0), a.Tm);   // clamped: see fwd.hip
  const int32_t* idx = a.col_idx + ((int64_t)bh * a.Tn + j) * a.Tm;
  if (parts) {                // entries [part * part_len, (part + 1) * part_len) of the list
    idx += part * part_len;
    cnt = min(cnt - part * part_len, part_len);
  }

  const int key0 = j * BKV + r32;                    // this lane's key of half 0; half 1 is 32 further

  if (cnt == 0) {   // no query block selected this key block: zero gradients (wave w writes key half w)
    const int key = key0 + 32 * w;
    if (key < N) {
      const int64_t out_off = base + (int64_t)key * a.sn + 4 * hf;
#pragma unroll
      for (int c = 0; c < D / 8; ++c) {
        *(u32x2*)(a.dk + out_off + 8 * c) = u32x2{0, 0};
        *(u32x2*)(a.dv + out_off + 8 * c) = u32x2{0, 0};
      }
    }
    return;
  }

  // K^T / V^T fragments (B operands): lane = key, 8 consecutive channels per 16-wide k step.  (Keys past N, in a short
  // last key block, repeat the last token: a key's column of every product is its own, and theirs are not stored.)
  bf16x8 kf[2][NK], vf[2][NK];
#pragma unroll
  for (int kh = 0; kh < 2; ++kh) {
    const int64_t off = base + (int64_t)min(key0 + 32 * kh, N - 1) * a.sn + 8 * hf;
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
      kf[kh][kk] = *(const bf16x8*)(a.k + off + 16 * kk);
      vf[kh][kk] = *(const bf16x8*)(a.v + off + 16 * kk);
    }
  }

  f32x16 dk_acc[2][NMB], dv_acc[2][NMB];
#pragma unroll
  for (int kh = 0; kh < 2; ++kh)
#pragma unroll
    for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
      for (int v = 0; v < 16; ++v) { dk_acc[kh][mb][v] = 0.f; dv_acc[kh][mb][v] = 0.f; }

  // global -> LDS copies of this wave's 32 rows.  A wave-wide 16-byte-per-lane copy lands linearly (wave base +
  // 16 * lane), i.e. lane l fills chunk position l % CPR of row RPI * r + l / CPR for copy instruction r; the
  // swizzle is applied on the source side (the lane fetches logical chunk position ^ swz(row)).  Everything else of a
  // request is wave-uniform: one 64-bit base per tensor and step and compile-time LDS offsets.  Rows past N (32 rows
  // that reach past the last token) are clamped to the last token, in the lane offsets, which are computed again only
  // when the number of valid rows changes.
  uint32_t voff[NCP], soff = 0;
  int rows_set = -1;
  auto set_rows = [&](int last) {            // last: last valid row of the 32 (uniform)
    if (last == rows_set) return;
    rows_set = last;
    const int l = fresh_lane();
#pragma unroll
    for (int r = 0; r < NCP; ++r) {
      const int row_l = RPI * r + l / CPR;
      voff[r] = (uint32_t)((min(row_l, last) * a.sn + (((l % CPR) ^ swz<D>(row_l)) * 8)) * 2);
    }
    soff = (uint32_t)(min(l & 31, last) * 4);
  };
  const char* q_head = (const char*)(a.q + base);
  const char* o_head = (const char*)(a.d_o + base);
  const char* lse_head = (const char*)(a.lse + (int64_t)bh * N);
  const char* dlt_head = (const char*)(a.delta + (int64_t)bh * N);
  const uint64_t row_bytes = (uint64_t)a.sn * 2;
  const uint32_t wsm = lds_addr_of(smem) + 2 * w * STAGE_B;       // uniform LDS byte addresses
  const uint32_t wstat = lds_addr_of(stat_s) + 2 * w * STAT_B;
  auto copy_stats = [&](int row, uint32_t stat_addr) {
    raw_copy4_to_lds_at<0>(lse_head + (uint64_t)row * 4, soff, stat_addr);
    raw_copy4_to_lds_at<256>(dlt_head + (uint64_t)row * 4, soff, stat_addr);
  };
  // Query rows past N get an LSE of +infinity once their copy has landed: their P is then exactly zero.
  auto mark_rows_past_end = [&](int row0, uint32_t stat_addr) {
    if (row0 + QW <= N) return;
    const int row_l = fresh_lane() & 31;
    if (row0 + row_l >= N) lds_stf(stat_addr + 4 * row_l, INFINITY);
  };

  // the index list, 64 entries at a time in one register (lane l holds entry 64c + l): reading entry t is a
  // lane read, not a memory access
  int idx_v = idx[min(lane, cnt - 1)];
  auto step_row = [&](int u) -> int {        // first row of step u (uniform, inside the chunk that idx_v holds)
    const int i = min(max(__builtin_amdgcn_readlane(idx_v, (u >> 1) & 63), 0), a.Tm - 1);
    return i * BQ + (u & 1) * HQ + QW * w;
  };

  // per-lane LDS byte offsets inside a 32-row tile.  Row reads: row r32, logical chunk 2kk + hf (the part that
  // depends on kk is XORed in as kk << 5).  Transposing reads: row 16c + 8*which + 4hf + (s16>>2), columns
  // 32mb + 16hb + 4(s16&3) (the part that depends on mb is XORed in as mb << 6).
  const int s16 = lane & 15, hb16 = (lane >> 4) & 1;
  const uint32_t a_off = 2 * swz_idx<D>(r32, 8 * hf);
  const uint32_t t_off0 = 2 * swz_idx<D>(4 * hf + (s16 >> 2), 16 * hb16 + 4 * (s16 & 3));
  const uint32_t t_off1 = 2 * swz_idx<D>(8 + 4 * hf + (s16 >> 2), 16 * hb16 + 4 * (s16 & 3));

  const int steps = 2 * cnt;                 // step u: half u & 1 of list entry u >> 1
  {
    const int row0 = step_row(0), row_b = min(row0, N - 1);
    set_rows(min(QW - 1, N - 1 - row_b));
    copy_stats(row_b, wstat);
    static_for<0, NCP>([&](auto R) {
      constexpr int r = decltype(R)::v;
      raw_copy16_to_lds_at<r * 1024>(q_head + (uint64_t)row_b * row_bytes, voff[r], wsm);
      raw_copy16_to_lds_at<TILE_B + r * 1024>(o_head + (uint64_t)row_b * row_bytes, voff[r], wsm);
    });
    raw_copies_done();
    mark_rows_past_end(row0, wstat);
  }
  // -V^T: the dP products then give -dO V^T on top of D, so that dS = P (dP - D) needs no subtraction (the sign of dS
  // is taken back with the scale of dK)
#pragma unroll
  for (int kh = 0; kh < 2; ++kh)
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) vf[kh][kk] = __builtin_bit_cast(bf16x8, __builtin_bit_cast(u32x4, vf[kh][kk]) ^ 0x80008000u);

  constexpr int PD = 4;                      // how many row fragments ahead an LDS read is issued
  constexpr int NX = 2 * NMB, PDT = 2;       // transposed fragments of a tile, and how many ahead they are read
  constexpr int EB = D == 128 ? 10 : 8;      // exp units (below) that run between the dP products
  bf16x8 fr[PD];
#pragma unroll
  for (int x = 0; x < PD; ++x) fr[x] = lds_ld16((wsm + a_off) ^ (x << 5));

  for (int u = 0; u < steps; ++u) {
    const int st = u & 1;
    const int un = min(u + 1, steps - 1);    // past the end the last step is requested again (nobody reads it)
    if (((u + 1) & 127) == 0 && u + 1 < steps) idx_v = list_load(idx, min(((u + 1) >> 1) + fresh_lane(), cnt - 1));   // next 64 entries
    const int row_nx = step_row(un), row_b = min(row_nx, N - 1);
    set_rows(min(QW - 1, N - 1 - row_b));
    const uint32_t nx_stage = wsm + (st ^ 1) * STAGE_B, nx_stat = wstat + (st ^ 1) * STAT_B;
    const char* qn = q_head + (uint64_t)row_b * row_bytes;
    const char* on = o_head + (uint64_t)row_b * row_bytes;
    // this step's operand addresses (one add per step; the XOR of the compile-time part is one more op per read)
    const uint32_t q_rd = wsm + st * STAGE_B + a_off, q_t0 = wsm + st * STAGE_B + t_off0, q_t1 = wsm + st * STAGE_B + t_off1;
    const uint32_t lb = wstat + st * STAT_B + 16 * hf;
    uint32_t lb1 = lb;
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+v"(lb1));            // (D is read into both key halves' accumulators, not read once and copied)
#endif

    // fragment y of the sequence is Q chunk y (y < NK) or dO chunk y - NK
    auto row_frag = [&](int y) -> bf16x8 { return lds_ld16((q_rd ^ ((y % NK) << 5)) + (y < NK ? 0 : TILE_B)); };
    auto tr_frag = [&](int tile, int x) -> bf16x8 {     // tile 0 = Q, 1 = dO; x = c * NMB + mb
      const int c = x / NMB, mb = x % NMB;
      const uint32_t o = tile * TILE_B + 32 * c * D;
      return join_tr(lds_tr4_at((q_t0 ^ (mb << 6)) + o), lds_tr4_at((q_t1 ^ (mb << 6)) + o));
    };
    f32x16 s[2], dp[2];
    f32x4 l_raw, l_neg;
    uint32_t pk[2][8], dsk[2][8];
    // exp unit e: two queries of accumulator group g = e / 4 (registers 4g .. 4g+3), key half (e / 2) % 2
    auto exp_unit = [&](auto E) {
      constexpr int e = decltype(E)::v, g = e >> 2, kh = (e >> 1) & 1, v = 4 * g + 2 * (e & 1);
      if constexpr ((e & 3) == 0) {
#pragma unroll
        for (int x = 0; x < 4; ++x) l_neg[x] = -LOG2E * l_raw[x];
        if constexpr (g < 3) l_raw = lds_ldf4(lb + 32 * (g + 1));
      }
      s[kh][v] = fast_exp2(fmaf(s[kh][v], a.scale_log2, l_neg[v & 3]));
      s[kh][v + 1] = fast_exp2(fmaf(s[kh][v + 1], a.scale_log2, l_neg[(v & 3) + 1]));
      pk[kh][v >> 1] = pack_bf16(s[kh][v], s[kh][v + 1]);
    };
    auto ds_unit = [&](auto E) {             // the same two queries of -dS = P * (D - dP)
      constexpr int e = decltype(E)::v, g = e >> 2, kh = (e >> 1) & 1, v = 4 * g + 2 * (e & 1);
      dsk[kh][v >> 1] = pack_bf16(s[kh][v] * dp[kh][v], s[kh][v + 1] * dp[kh][v + 1]);
    };
    auto quad = [](const uint32_t (&p)[8], int c) -> bf16x8 {
      return __builtin_bit_cast(bf16x8, u32x4{p[4 * c], p[4 * c + 1], p[4 * c + 2], p[4 * c + 3]});
    };

    // ---- S = Q K^T; the next step's LSE, D and Q rows are requested
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    static_for<0, NK>([&](auto Y) {
      constexpr int y = decltype(Y)::v;
      s[0] = mfma32(fr[y % PD], kf[0][y], y == 0 ? zero : s[0]);
      s[1] = mfma32(fr[y % PD], kf[1][y], y == 0 ? zero : s[1]);
      if constexpr (y == 0) copy_stats(row_b, nx_stat);
      raw_copy16_to_lds_at<y * 1024>(qn, voff[y], nx_stage);
      if constexpr (y + PD == NK) raw_copies_left<2 + y + 1>();      // this step's dO rows have landed
      fr[y % PD] = row_frag(y + PD);
      if constexpr (y >= NK - 4) {           // D, as the initial value of dP
        constexpr int g = y - (NK - 4);
        const f32x4 d0 = lds_ldf4(lb + 256 + 32 * g), d1 = lds_ldf4(lb1 + 256 + 32 * g);
#pragma unroll
        for (int x = 0; x < 4; ++x) { dp[0][4 * g + x] = d0[x]; dp[1][4 * g + x] = d1[x]; }
      }
      if constexpr (y == NK - 1) l_raw = lds_ldf4(lb);
      __builtin_amdgcn_sched_barrier(0);
    });
    // ---- D - dP = D + dO (-V)^T, with exp(S - LSE) between the products; the next step's dO rows are requested
    bf16x8 ft[PDT];
    static_for<0, NK>([&](auto Y) {
      constexpr int y = decltype(Y)::v;
      dp[0] = mfma32(fr[y % PD], vf[0][y], dp[0]);
      dp[1] = mfma32(fr[y % PD], vf[1][y], dp[1]);
      if constexpr (y + PD < NK) fr[y % PD] = row_frag(NK + y + PD);
      raw_copy16_to_lds_at<TILE_B + y * 1024>(on, voff[y], nx_stage);
      static_for<y * EB / NK, (y + 1) * EB / NK>(exp_unit);
      if constexpr (y >= NK - PDT) ft[y - (NK - PDT)] = tr_frag(1, y - (NK - PDT));
      __builtin_amdgcn_sched_barrier(0);
    });
    // ---- dV^T += dO^T P.  Step x = (c, mb): the 16 queries 16c.. (accumulator registers 8c .. 8c+7), output block mb;
    // each transposed fragment feeds both key halves.  The remaining exponentials run between the first half of the
    // products, dS of the first 16 queries between the second.
    static_for<0, NX>([&](auto X) {
      constexpr int x = decltype(X)::v, c = x / NMB, mb = x % NMB;
      mfma32_acc(ft[x % PDT], quad(pk[0], c), dv_acc[0][mb]);
      mfma32_acc(ft[x % PDT], quad(pk[1], c), dv_acc[1][mb]);
      ft[x % PDT] = x + PDT < NX ? tr_frag(1, x + PDT) : tr_frag(0, x + PDT - NX);
      if constexpr (c == 0) static_for<EB + mb * (16 - EB) / NMB, EB + (mb + 1) * (16 - EB) / NMB>(exp_unit);
      else                  static_for<mb * 8 / NMB, (mb + 1) * 8 / NMB>(ds_unit);
      __builtin_amdgcn_sched_barrier(0);
    });
    // ---- -dK^T += Q^T (-dS), the same way, with dS of the other 16 queries between the first half; then the next
    // step's Q rows, LSE and D have landed (its dO rows, the last NCP copies, may be in flight) and its first row
    // fragments are read
    static_for<0, NX>([&](auto X) {
      constexpr int x = decltype(X)::v, c = x / NMB, mb = x % NMB;
      mfma32_acc(ft[x % PDT], quad(dsk[0], c), dk_acc[0][mb]);
      mfma32_acc(ft[x % PDT], quad(dsk[1], c), dk_acc[1][mb]);
      if constexpr (x + PDT < NX) ft[x % PDT] = tr_frag(0, x + PDT);
      if constexpr (c == 0) static_for<8 + mb * 8 / NMB, 8 + (mb + 1) * 8 / NMB>(ds_unit);
      if constexpr (x == NMB) {
        raw_copies_left<NCP>();
        mark_rows_past_end(row_nx, nx_stat);
      }
      if constexpr (c == 1) {
#pragma unroll
        for (int f = mb * PD / NMB; f < (mb + 1) * PD / NMB; ++f) fr[f] = lds_ld16((nx_stage + a_off) ^ (f << 5));
      }
      __builtin_amdgcn_sched_barrier(0);
    });
  }

  // the accumulators are read by ordinary vector instructions from here on: let the last products finish first
  // (the compiler does not know that mfma32_acc is a matrix instruction and inserts no wait states for it); and the
  // copies of the step past the end have to be out of the way of the exchange below
  raw_copies_done();
  walk.draw(a.sp);
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
#endif
  // The two waves' partial sums are added: wave w hands its sums of key half 1 - w over, through its own staging area,
  // and finishes key half w.  16-byte pieces [tensor][output block][group][lane], one exchange for both tensors (two of
  // all sums before, four bytes at a time: with the order of the step above, 54 -> 47 us for 504 columns of 4 entries).
  constexpr int REGION = 2 * NMB * 4 * 64 * 4;        // floats per wave
  static_assert(REGION * 4 == 2 * STAGE_B, "the sums that a wave hands over fill exactly its two stages");
  float* scratch = (float*)smem;
  const int le = fresh_lane(), he = le >> 5, key0w = j * BKV + 32 * w;        // first of the keys that this wave finishes
  auto hand_over = [&](auto KH) {
    f32x4* out = (f32x4*)(scratch + w * REGION) + le;
    static_for<0, 8 * NMB>([&](auto C) {
      constexpr int c = decltype(C)::v, mb = (c / 4) % NMB, v = 4 * (c % 4);
      const f32x16& x = c < 4 * NMB ? dk_acc[decltype(KH)::v][mb] : dv_acc[decltype(KH)::v][mb];
      out[64 * c] = f32x4{x[v], x[v + 1], x[v + 2], x[v + 3]};
      if constexpr (c % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    });
  };
  // put(tensor, output block, group, sums) of every piece that this wave finishes
  auto finish = [&](auto KH, auto&& put) {
    const f32x4* in = (const f32x4*)(scratch + (1 - w) * REGION) + le;
    static_for<0, 8 * NMB>([&](auto C) {
      constexpr int c = decltype(C)::v, mb = (c / 4) % NMB, v = 4 * (c % 4);
      const f32x16& x = c < 4 * NMB ? dk_acc[decltype(KH)::v][mb] : dv_acc[decltype(KH)::v][mb];
      put(c / (4 * NMB), mb, c % 4, f32x4{x[v], x[v + 1], x[v + 2], x[v + 3]} + in[64 * c]);
      if constexpr (c % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    });
  };
  if (w == 0) hand_over(Int<1>{});
  else        hand_over(Int<0>{});
  __syncthreads();
  if (parts) {                  // one part of a split column: leave the sums to the last part (the whole slot is
    float* ps = a.sp.pool + (int64_t)item.slot * a.sp.slot_floats + 2 * le;       // written: the merge reads it)
    auto put = [&](int t, int mb, int g, f32x4 x) {
      float* p = ps + (((t * 2 + w) * NMB + mb) * 4 + g) * 256;
      part_store2(p, x[0], x[1]);
      part_store2(p + 128, x[2], x[3]);
    };
    if (w == 0) finish(Int<0>{}, put);
    else        finish(Int<1>{}, put);
  } else {
    u32x2 done[8 * NMB];
    auto put = [&](int t, int mb, int g, f32x4 x) {
      const float sc = t == 0 ? -a.scale : 1.f;
      done[(t * NMB + mb) * 4 + g] = u32x2{pack_bf16(x[0] * sc, x[1] * sc), pack_bf16(x[2] * sc, x[3] * sc)};
    };
    if (w == 0) finish(Int<0>{}, put);
    else        finish(Int<1>{}, put);
    // (the sums that this wave has just read are what the other one handed over: their place is free)
    const uint32_t area = lds_addr_of(scratch + (1 - w) * REGION);
    static_for<0, 8 * NMB>([&](auto C) {
      constexpr int c = decltype(C)::v;
      row_piece_put<D>(area + (c / (4 * NMB)) * (32 * D * 2), le & 31, c % (4 * NMB), he, done[c]);
    });
    rows_store<D>(area, a.dk + base + (int64_t)key0w * a.sn, a.sn, N - key0w, le);
    rows_store<D>(area + 32 * D * 2, a.dv + base + (int64_t)key0w * a.sn, a.sn, N - key0w, le);
    return;
  }
  if (!last_part(a.sp.arrive + item.slot - part, parts, (int*)stat_s)) return;
  dkdv_merge<D>(a, item, base, key0w, w, le, lds_addr_of(scratch + w * REGION));
}

// Head dimension 64: one workgroup of two waves per key block, two waves per SIMD (256 registers), eight per CU.  Wave w owns
// keys 32w .. 32w + 31 and all 64 query rows of a step, in two halves of 32; K^T, V^T (32 registers) and the sums (64) stay
// in registers.  An operand fragment from LDS feeds one product instead of the two of dkdv_item, but the sums need no
// exchange at the end, and a second wave on the SIMD works where this one waits: the exponentials per product are twice
// those of d = 128, a single wave kept the matrix cores busy 39 % of the time.  Rows are staged once for both waves (each
// copies 32 of them, a step ahead), one barrier a step.
//   S rh = Q K^T, rh = 0, 1   | copies of the next step; D into the accumulators of dP 0
//   D - dP 0, D - dP 1        | exponentials of half 0, of half 1
//   dV of half 0, of half 1   | dS of half 0, of half 1
//   dK of half 0, of half 1   | barrier, first fragments of the next step
// Bound: the copies out of the memory-side cache (9 TB/s over all compute units while every slot is busy).  Measured, us, a
// training pass, one wave a SIMD with 64 keys a wave / this: 20,010 tokens, 6 heads 280 / 270; 40,296 tokens, 32 heads
// 4202 / 3983.  256 columns of 4 entries, a workgroup a compute unit: 20.0 / 19.5 (the kernel).
__device__ __forceinline__ void dkdv_item64(const DkvArgs& a, const WorkItem& item, Walk& walk, unsigned char* smem,
                                            unsigned char* stat_s) {
  constexpr int D = 64, NK = D / 16, NMB = D / 32;
  constexpr int HQ = 64;                             // query rows per step
  constexpr int CPR = D / 8, RPI = 64 / CPR, NCP = 32 / RPI;         // (see dkdv_item)
  constexpr int TILE_B = HQ * D * 2, HALF_B = TILE_B / 2, STAGE_B = 2 * TILE_B;    // Q rows, then dO rows
  constexpr int STAT_B = 512;                        // a wave's 32 rows: LSE at +0, D at +256
  const int bh = item.bh, j = item.blk, part = item.part, parts = item.parts, part_len = item.part_len;
  const int64_t base = (int64_t)(bh / a.H) * a.sb + (int64_t)(bh % a.H) * a.sh;
  const int lane = fresh_lane(), w = walk.wave;
  const int r32 = lane & 31, hf = lane >> 5;
  const int N = a.N;
  int cnt = min(max(a.col_cnt[(int64_t)bh * a.Tn + j], 0), a.Tm);   // clamped: see fwd.hip
  const int32_t* idx = a.col_idx + ((int64_t)bh * a.Tn + j) * a.Tm;
  if (parts) {                // entries [part * part_len, (part + 1) * part_len) of the list
    idx += part * part_len;
    cnt = min(cnt - part * part_len, part_len);
  }
  const int key0w = j * BKV + 32 * w, key = key0w + r32;
  if (cnt == 0) {             // no query block selected this key block: zero gradients
    if (key < N) {
      const int64_t out_off = base + (int64_t)key * a.sn + 32 * hf;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        *(u32x4*)(a.dk + out_off + 8 * c) = u32x4{0, 0, 0, 0};
        *(u32x4*)(a.dv + out_off + 8 * c) = u32x4{0, 0, 0, 0};
      }
    }
    return;
  }

  // K^T / V^T fragments: lane = key, 8 consecutive channels per 16-wide k step (keys past N repeat the last token)
  bf16x8 kf[NK], vf[NK];
  {
    const int64_t off = base + (int64_t)min(key, N - 1) * a.sn + 8 * hf;
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
      kf[kk] = *(const bf16x8*)(a.k + off + 16 * kk);
      vf[kk] = *(const bf16x8*)(a.v + off + 16 * kk);
    }
  }
  f32x16 dk_acc[NMB], dv_acc[NMB];
#pragma unroll
  for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
    for (int v = 0; v < 16; ++v) { dk_acc[mb][v] = 0.f; dv_acc[mb][v] = 0.f; }

  // copies of rows 32w .. 32w + 31 of a step (swizzled and clamped as in dkdv_item)
  uint32_t voff[NCP], soff = 0;
  int rows_set = -1;
  auto set_rows = [&](int last) {            // last: last valid row of the 32 (uniform)
    if (last == rows_set) return;
    rows_set = last;
    const int l = fresh_lane();
#pragma unroll
    for (int r = 0; r < NCP; ++r) {
      const int row_l = RPI * r + l / CPR;
      voff[r] = (uint32_t)((min(row_l, last) * a.sn + (((l % CPR) ^ swz<D>(row_l)) * 8)) * 2);
    }
    soff = (uint32_t)(min(l & 31, last) * 4);
  };
  const char* q_head = (const char*)(a.q + base);
  const char* o_head = (const char*)(a.d_o + base);
  const char* lse_head = (const char*)(a.lse + (int64_t)bh * N);
  const char* dlt_head = (const char*)(a.delta + (int64_t)bh * N);
  const uint64_t row_bytes = (uint64_t)a.sn * 2;
  const uint32_t sm = lds_addr_of(smem), stat = lds_addr_of(stat_s);
  const uint32_t sm_w = sm + w * HALF_B, stat_w = stat + w * STAT_B;         // this wave's rows of a stage
  auto copy_stats = [&](int row, uint32_t stat_addr) {
    raw_copy4_to_lds_at<0>(lse_head + (uint64_t)row * 4, soff, stat_addr);
    raw_copy4_to_lds_at<256>(dlt_head + (uint64_t)row * 4, soff, stat_addr);
  };
  // Query rows past N get an LSE of +infinity once their copy has landed: their P is then exactly zero.
  auto mark_rows_past_end = [&](int row0, uint32_t stat_addr) {
    if (row0 + 32 <= N) return;
    const int row_l = fresh_lane() & 31;
    if (row0 + row_l >= N) lds_stf(stat_addr + 4 * row_l, INFINITY);
  };

  int idx_v = idx[min(lane, cnt - 1)];       // the index list, 64 entries at a time (see dkdv_item)
  auto step_row = [&](int u) -> int {        // this wave's first row of step u (uniform, inside the chunk that idx_v holds)
    const int i = min(max(__builtin_amdgcn_readlane(idx_v, (u >> 1) & 63), 0), a.Tm - 1);
    return i * BQ + (u & 1) * HQ + 32 * w;
  };
  const int s16 = lane & 15, hb16 = (lane >> 4) & 1;
  const uint32_t a_off = sm + 2 * swz_idx<D>(r32, 8 * hf);
  const uint32_t t_off0 = sm + 2 * swz_idx<D>(4 * hf + (s16 >> 2), 16 * hb16 + 4 * (s16 & 3));
  const uint32_t t_off1 = sm + 2 * swz_idx<D>(8 + 4 * hf + (s16 >> 2), 16 * hb16 + 4 * (s16 & 3));

  const int steps = 2 * cnt;                 // step u: half u & 1 of list entry u >> 1
  {
    const int row0 = step_row(0), row_b = min(row0, N - 1);
    set_rows(min(31, N - 1 - row_b));
    copy_stats(row_b, stat_w);
    static_for<0, NCP>([&](auto R) {
      constexpr int r = decltype(R)::v;
      raw_copy16_to_lds_at<r * 1024>(q_head + (uint64_t)row_b * row_bytes, voff[r], sm_w);
      raw_copy16_to_lds_at<TILE_B + r * 1024>(o_head + (uint64_t)row_b * row_bytes, voff[r], sm_w);
    });
    raw_copies_done();
    mark_rows_past_end(row0, stat_w);
    __syncthreads();
  }
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) vf[kk] = __builtin_bit_cast(bf16x8, __builtin_bit_cast(u32x4, vf[kk]) ^ 0x80008000u);   // -V^T (see dkdv_item)

  constexpr int PD = 4, PDT = 2;             // how many row / transposed fragments ahead an LDS read is issued
  constexpr int NR = 2 * NK, NX = 4 * NMB;   // row fragments of one tensor and step; transposed ones (rh, c, mb)
  bf16x8 fr[PD];
  auto row_frag = [&](uint32_t at, int y) -> bf16x8 {         // y = (tensor, rh, kk)
    return lds_ld16((at ^ ((y % NK) << 5)) + (y / NR) * TILE_B + ((y / NK) % 2) * HALF_B);
  };
#pragma unroll
  for (int x = 0; x < PD; ++x) fr[x] = row_frag(a_off, x);

  for (int u = 0; u < steps; ++u) {
    const int st = u & 1;
    const int un = min(u + 1, steps - 1);    // past the end the last step is requested again (nobody reads it)
    if (((u + 1) & 127) == 0 && u + 1 < steps) idx_v = list_load(idx, min(((u + 1) >> 1) + fresh_lane(), cnt - 1));   // next 64 entries
    const int row_nx = step_row(un), row_b = min(row_nx, N - 1);
    set_rows(min(31, N - 1 - row_b));
    const uint32_t nx_stage = sm_w + (st ^ 1) * STAGE_B, nx_stat = stat_w + (st ^ 1) * 2 * STAT_B;
    const char* qn = q_head + (uint64_t)row_b * row_bytes;
    const char* on = o_head + (uint64_t)row_b * row_bytes;
    uint32_t q_rd = a_off + st * STAGE_B, q_t0 = t_off0 + st * STAGE_B, q_t1 = t_off1 + st * STAGE_B;
    const uint32_t lb = stat + st * 2 * STAT_B + 16 * hf;
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+v"(q_rd), "+v"(q_t0), "+v"(q_t1));    // (the XORed addresses are not kept over the loop)
#endif
    auto tr_frag = [&](int tile, int x) -> bf16x8 {     // tile 0 = Q, 1 = dO; x = (rh, c, mb)
      const uint32_t o = tile * TILE_B + (x / NMB) * 32 * D;
      return join_tr(lds_tr4_at((q_t0 ^ ((x % NMB) << 6)) + o), lds_tr4_at((q_t1 ^ ((x % NMB) << 6)) + o));
    };
    f32x16 s[2], dp[2];
    f32x4 l_raw, l_neg;
    uint32_t pk[2][8], dsk[2][8];
    auto load_d = [&](int rh) {              // D, as the initial value of dP
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x4 d0 = lds_ldf4(lb + 256 + STAT_B * rh + 32 * g);
#pragma unroll
        for (int x = 0; x < 4; ++x) dp[rh][4 * g + x] = d0[x];
      }
    };
    // exp unit e = (rh, g, pair): two queries of accumulator group g (registers 4g .. 4g+3)
    auto exp_unit = [&](auto E) {
      constexpr int e = decltype(E)::v, rh = e >> 3, g = (e >> 1) & 3, v = 4 * g + 2 * (e & 1);
      if constexpr ((e & 1) == 0) {
#pragma unroll
        for (int x = 0; x < 4; ++x) l_neg[x] = -LOG2E * l_raw[x];
        if constexpr (e < 14) l_raw = lds_ldf4(lb + STAT_B * ((e + 2) >> 3) + 32 * (((e + 2) >> 1) & 3));
      }
      s[rh][v] = fast_exp2(fmaf(s[rh][v], a.scale_log2, l_neg[v & 3]));
      s[rh][v + 1] = fast_exp2(fmaf(s[rh][v + 1], a.scale_log2, l_neg[(v & 3) + 1]));
      pk[rh][v >> 1] = pack_bf16(s[rh][v], s[rh][v + 1]);
    };
    auto ds_unit = [&](auto E) {             // the same two queries of -dS = P * (D - dP)
      constexpr int e = decltype(E)::v, rh = e >> 3, v = 4 * ((e >> 1) & 3) + 2 * (e & 1);
      dsk[rh][v >> 1] = pack_bf16(s[rh][v] * dp[rh][v], s[rh][v + 1] * dp[rh][v + 1]);
    };
    auto quad = [](const uint32_t (&p)[8], int c) -> bf16x8 {
      return __builtin_bit_cast(bf16x8, u32x4{p[4 * c], p[4 * c + 1], p[4 * c + 2], p[4 * c + 3]});
    };
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    // ---- S = Q K^T of both halves; the next step's LSE, D, Q and dO rows are requested
    static_for<0, NR>([&](auto Y) {
      constexpr int y = decltype(Y)::v, rh = y / NK, kk = y % NK;
      s[rh] = mfma32(fr[y % PD], kf[kk], kk == 0 ? zero : s[rh]);
      fr[y % PD] = row_frag(q_rd, y + PD);
      if constexpr (y == 0) copy_stats(row_b, nx_stat);
      if constexpr (y < NCP) raw_copy16_to_lds_at<y * 1024>(qn, voff[y], nx_stage);
      else                   raw_copy16_to_lds_at<TILE_B + (y - NCP) * 1024>(on, voff[y - NCP], nx_stage);
      if constexpr (y == NK) load_d(0);
      if constexpr (y == NR - 1) l_raw = lds_ldf4(lb);
      __builtin_amdgcn_sched_barrier(0);
    });
    // ---- D - dP = D + dO (-V)^T, with exp(S - LSE) between the products
    bf16x8 ft[PDT];
    static_for<0, NR>([&](auto Y) {
      constexpr int y = decltype(Y)::v, rh = y / NK, kk = y % NK;
      dp[rh] = mfma32(fr[y % PD], vf[kk], dp[rh]);
      if constexpr (y + PD < NR) fr[y % PD] = row_frag(q_rd, NR + y + PD);
      if constexpr (y == 0) load_d(1);
      static_for<y * 2, y * 2 + 2>(exp_unit);
      if constexpr (y >= NR - PDT) ft[y - (NR - PDT)] = tr_frag(1, y - (NR - PDT));
      __builtin_amdgcn_sched_barrier(0);
    });
    // ---- dV^T += dO^T P.  Step x = (rh, c, mb): the 16 queries 16c.. of half rh, output block mb
    static_for<0, NX>([&](auto X) {
      constexpr int x = decltype(X)::v, mb = x % NMB, c = (x / NMB) % 2, rh = x / (2 * NMB);
      dv_acc[mb] = mfma32(ft[x % PDT], quad(pk[rh], c), dv_acc[mb]);
      ft[x % PDT] = x + PDT < NX ? tr_frag(1, x + PDT) : tr_frag(0, x + PDT - NX);
      static_for<x * 2, x * 2 + 2>(ds_unit);
      __builtin_amdgcn_sched_barrier(0);
    });
    // ---- -dK^T += Q^T (-dS).  When the last fragments of this step have been read and the next step's rows have landed,
    // both waves change stages
    static_for<0, NX>([&](auto X) {
      constexpr int x = decltype(X)::v, mb = x % NMB, c = (x / NMB) % 2, rh = x / (2 * NMB);
      dk_acc[mb] = mfma32(ft[x % PDT], quad(dsk[rh], c), dk_acc[mb]);
      if constexpr (x + PDT < NX) ft[x % PDT] = tr_frag(0, x + PDT);
      if constexpr (x == NX - PDT) {
        raw_copies_done();
        mark_rows_past_end(row_nx, nx_stat);
        __syncthreads();
#pragma unroll
        for (int f = 0; f < PD; ++f) fr[f] = row_frag(a_off + (st ^ 1) * STAGE_B, f);
      }
      __builtin_amdgcn_sched_barrier(0);
    });
  }
  walk.draw(a.sp);
  // The stage that nobody was to read has landed (the barrier of the last step): its LDS, and with one more barrier the
  // other stage's, is free.
  const int le = fresh_lane();
  if (parts) {                  // one part of a split column: leave the sums to the last part
    float* ps = a.sp.pool + (int64_t)item.slot * a.sp.slot_floats + 2 * le;
    static_for<0, 2 * NMB * 8>([&](auto C) {
      constexpr int c = decltype(C)::v, t = c / (8 * NMB), mb = (c / 8) % NMB, v = 2 * (c % 8);
      const f32x16& x = t == 0 ? dk_acc[mb] : dv_acc[mb];
      part_store2(ps + ((t * 2 + w) * NMB * 8 + c % (8 * NMB)) * 128, x[v], x[v + 1]);
    });
    if (!last_part(a.sp.arrive + item.slot - part, parts, (int*)stat_s)) return;
    dkdv_merge<D>(a, item, base, key0w, w, le, sm + w * TILE_B);
    return;
  }
  __syncthreads();
  const uint32_t area = sm + w * TILE_B;             // dK, then dV rows of this wave
  static_for<0, 2 * NMB * 4>([&](auto C) {
    constexpr int c = decltype(C)::v, t = c / (4 * NMB), mb = (c / 4) % NMB, v = 4 * (c % 4);
    const f32x16& x = t == 0 ? dk_acc[mb] : dv_acc[mb];
    const float sc = t == 0 ? -a.scale : 1.f;
    row_piece_put<D>(area + t * (32 * D * 2), le & 31, c % (4 * NMB), le >> 5,
                     u32x2{pack_bf16(x[v] * sc, x[v + 1] * sc), pack_bf16(x[v + 2] * sc, x[v + 3] * sc)});
  });
  rows_store<D>(area, a.dk + base + (int64_t)key0w * a.sn, a.sn, N - key0w, le);
  rows_store<D>(area + 32 * D * 2, a.dv + base + (int64_t)key0w * a.sn, a.sn, N - key0w, le);
}

template <int D>
__global__ __attribute__((amdgpu_flat_work_group_size(128, 128), amdgpu_waves_per_eu(D == 128 ? 1 : 2, D == 128 ? 1 : 2)))
void dkdv_kernel(DkvArgs) {
  // two stages of 64 rows of Q and dO (aligned: compile-time parts are XORed into addresses)
  __shared__ __align__(1024) unsigned char smem[2 * 2 * 64 * D * 2];
  __shared__ __align__(1024) unsigned char stat_s[2 * 2 * 512];
  __shared__ int word;
  Walk walk(&word, fresh_args<DkvArgs>().sp);
  if (walk.idle(fresh_args<DkvArgs>().sp)) return;
  for (;;) {
    const DkvArgs& a = fresh_args<DkvArgs>();
    WorkItem item;
    if (!walk.take(item, a.sp, a.Tn, a.chunk, a.BH, a.col_order)) return;
    if constexpr (D == 128) dkdv_item<D>(a, item, walk, smem, stat_s);
    else                    dkdv_item64(a, item, walk, smem, stat_s);
    if (!walk.advance(a.sp)) return;
  }
}

hipError_t launch_bwd_dkdv(const void* q, const void* k, const void* v, const void* d_o, const float* lse,
                           const float* delta, const Dims& m, const int32_t* col_cnt, const int32_t* col_idx,
                           const int32_t* col_order, float scale, void* dk, void* dv, const SplitPlan& plan,
                           hipStream_t stream) {
  DkvArgs a;
  a.q = (const uint16_t*)q; a.k = (const uint16_t*)k; a.v = (const uint16_t*)v; a.d_o = (const uint16_t*)d_o;
  a.lse = lse; a.delta = delta; a.dk = (uint16_t*)dk; a.dv = (uint16_t*)dv;
  a.col_cnt = col_cnt; a.col_idx = col_idx; a.col_order = col_order;
  a.BH = m.B * m.H; a.H = m.H; a.N = m.N; a.Tm = m.Tm; a.Tn = m.Tn; a.chunk = (m.Tn + 7) / 8;
  a.sb = m.sb; a.sh = m.sh; a.sn = m.sn;
  a.scale = scale; a.scale_log2 = scale * LOG2E;
  a.sp = plan;
  if (plan.pool_slots && !plan.planned) {
    const hipError_t e = launch_split_plan(col_cnt, (int64_t)m.B * m.H * m.Tn, m.Tm, SPLIT_DKDV, plan, stream);
    if (e != hipSuccess) return e;
  }
  const int columns = plan.stretches ? stretch_wgs(a.BH * a.Tn) : xcd_map_wgs(a.BH, a.Tn, a.chunk, SHORT_COLUMNS);
  const dim3 grid((unsigned)(plan.queue && !plan.queue_if_full ? plan.resident : plan.pool_slots + columns)), block(128);
  if (m.d == 128) hipLaunchKernelGGL(dkdv_kernel<128>, grid, block, 0, stream, a);
  else            hipLaunchKernelGGL(dkdv_kernel<64>, grid, block, 0, stream, a);
  return hipGetLastError();
}

}  // namespace spa2
