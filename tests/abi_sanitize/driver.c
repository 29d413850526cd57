/* Host-only exerciser of the argument checks of the spa2 C ABI, built with AddressSanitizer and
 * UndefinedBehaviorSanitizer on the host side (tests/test_abi_cpu.py compiles and runs it).  Every call below
 * must be rejected before anything is launched: the kernel launchers are replaced by stubs that abort. */
#include <math.h>
#include <stdio.h>
#include <stdlib.h>

#include "spa2.h"

static int failures = 0;
#define EXPECT(call, code)                                                                  \
  do {                                                                                      \
    int rc_ = (call);                                                                       \
    if (rc_ != (code)) { printf("line %d: got %d, expected %d\n", __LINE__, rc_, (code)); ++failures; } \
  } while (0)

static spa2_shape shape(int B, int H, int N, int d, int bq, int bkv, long long sn) {
  spa2_shape s;
  s.B = B; s.H = H; s.N = N; s.d = d; s.bq = bq; s.bkv = bkv;
  s.sn = sn ? sn : d; s.sh = (long long)N * s.sn; s.sb = (long long)H * s.sh;
  return s;
}

int main(void) {
  void* fake = (void*)0x1000;   /* 16-byte aligned, never dereferenced on a rejected call */
  void* odd = (void*)0x1004;
  spa2_pattern none = {0, 0, 0, 0, 0, 0, 0};
  spa2_pattern full = {(uint8_t*)fake, (int32_t*)fake, (int32_t*)fake, (int32_t*)fake, (int32_t*)fake, 0, 0};
  spa2_pattern half = {(uint8_t*)fake, (int32_t*)fake, (int32_t*)fake, (int32_t*)fake, 0, 0, 0};
  spa2_pattern rows_only = {(uint8_t*)fake, (int32_t*)fake, (int32_t*)fake, 0, 0, 0, 0};
  spa2_shape ok = shape(1, 2, 300, 128, 128, 64, 0);
  spa2_shape d96 = shape(1, 2, 300, 96, 128, 64, 0), bq64 = shape(1, 2, 300, 128, 64, 64, 0);
  spa2_shape n0 = shape(1, 2, 0, 128, 128, 64, 0), sn132 = shape(1, 2, 300, 128, 128, 64, 132);
  spa2_shape wide = shape(1, 1, 300, 128, 128, 64, (1 << 23) + 8);
  spa2_shape longrow = shape(1, 2, 64 * 8193, 64, 128, 64, 0);
  spa2_shape many = shape(1 << 12, 1 << 12, 20000, 64, 128, 64, 0);
  spa2_shape huge = shape(1, 1, 128, 128, 128, 64, 0);                /* B*H*N would overflow 64 bits if multiplied blindly */
  huge.B = huge.H = huge.N = 0x7fffffff;
  spa2_shape toolong = shape(1, 4, SPA2_STATIC_MAX_ROWS / 4 + 64, 128, 128, 64, 0);
  size_t big = (size_t)1 << 40;

  EXPECT(spa2_fwd(0, fake, fake, &ok, &full, 0.1f, fake, 0, (float*)fake, 0, 0, 0), SPA2_ERR_NULL);
  EXPECT(spa2_fwd(fake, fake, fake, 0, &full, 0.1f, fake, 0, (float*)fake, 0, 0, 0), SPA2_ERR_NULL);
  EXPECT(spa2_fwd(fake, fake, fake, &ok, &none, 0.1f, fake, 0, (float*)fake, 0, 0, 0), SPA2_ERR_NULL);
  EXPECT(spa2_fwd(odd, fake, fake, &ok, &full, 0.1f, fake, 0, (float*)fake, 0, 0, 0), SPA2_ERR_ALIGN);
  EXPECT(spa2_fwd(fake, fake, fake, &ok, &full, 0.0f, fake, 0, (float*)fake, 0, 0, 0), SPA2_ERR_RANGE);
  EXPECT(spa2_fwd(fake, fake, fake, &ok, &full, NAN, fake, 0, (float*)fake, 0, 0, 0), SPA2_ERR_RANGE);
  EXPECT(spa2_fwd(fake, fake, fake, &d96, &full, 0.1f, fake, 0, (float*)fake, 0, 0, 0), SPA2_ERR_UNSUPPORTED);
  EXPECT(spa2_fwd(fake, fake, fake, &bq64, &full, 0.1f, fake, 0, (float*)fake, 0, 0, 0), SPA2_ERR_UNSUPPORTED);
  EXPECT(spa2_fwd(fake, fake, fake, &n0, &full, 0.1f, fake, 0, (float*)fake, 0, 0, 0), SPA2_ERR_SHAPE);
  EXPECT(spa2_fwd(fake, fake, fake, &sn132, &full, 0.1f, fake, 0, (float*)fake, 0, 0, 0), SPA2_ERR_ALIGN);
  EXPECT(spa2_fwd(fake, fake, fake, &wide, &full, 0.1f, fake, 0, (float*)fake, 0, 0, 0), SPA2_ERR_SHAPE);
  EXPECT(spa2_fwd(fake, fake, fake, &many, &full, 0.1f, fake, 0, (float*)fake, 0, 0, 0), SPA2_ERR_SHAPE);
  EXPECT(spa2_fwd(fake, fake, fake, &huge, &full, 0.1f, fake, 0, (float*)fake, 0, 0, 0), SPA2_ERR_SHAPE);

  EXPECT(spa2_fwd(fake, fake, fake, &ok, &full, 0.1f, fake, 0, (float*)fake, odd, big, 0), SPA2_ERR_ALIGN);
  EXPECT(spa2_mask(fake, fake, &ok, 1, 0.5f, 0.1f, &full, 0, 0, big, 0), SPA2_ERR_WORKSPACE);
  EXPECT(spa2_mask(fake, fake, &ok, 1, 0.5f, 0.1f, &full, 0, fake, 16, 0), SPA2_ERR_WORKSPACE);
  EXPECT(spa2_mask(fake, fake, &ok, 0, 0.0f, 0.1f, &full, 0, fake, big, 0), SPA2_ERR_RANGE);
  EXPECT(spa2_mask(fake, fake, &ok, 6, 0.5f, 0.1f, &full, 0, fake, big, 0), SPA2_ERR_RANGE);
  EXPECT(spa2_mask(fake, fake, &ok, -1, 0.5f, 0.1f, &full, 0, fake, big, 0), SPA2_ERR_RANGE);
  EXPECT(spa2_mask(fake, fake, &ok, 1, 1.5f, 0.1f, &full, 0, fake, big, 0), SPA2_ERR_RANGE);
  EXPECT(spa2_mask(fake, fake, &ok, 1, NAN, 0.1f, &full, 0, fake, big, 0), SPA2_ERR_RANGE);
  EXPECT(spa2_mask(fake, fake, &longrow, 1, 0.5f, 0.1f, &full, 0, fake, big, 0), SPA2_ERR_SHAPE);
  EXPECT(spa2_mask(fake, fake, &ok, 1, 0.5f, 0.1f, &half, 0, fake, big, 0), SPA2_ERR_NULL);
  EXPECT(spa2_mask_pool(fake, fake, &ok, fake, 16, 0), SPA2_ERR_WORKSPACE);
  EXPECT(spa2_mask_select(&ok, 1, 0.5f, 0.1f, &none, 0, fake, big, 0), SPA2_ERR_NULL);
  EXPECT(spa2_mask_columns(&longrow, &full, 0), SPA2_ERR_SHAPE);
  EXPECT(spa2_mask_columns(&many, &full, 0), SPA2_ERR_SHAPE);
  EXPECT(spa2_mask_columns(&ok, &rows_only, 0), SPA2_ERR_NULL);
  EXPECT(spa2_pattern_full(&ok, 0, 0), SPA2_ERR_NULL);

  EXPECT(spa2_bwd(fake, fake, fake, fake, 0, fake, (float*)fake, &ok, &rows_only, 0.1f, fake, fake, fake, fake, big, 0),
         SPA2_ERR_NULL);
  EXPECT(spa2_bwd(fake, fake, fake, fake, 0, fake, (float*)fake, &ok, &full, 0.1f, fake, fake, fake, fake, 8, 0),
         SPA2_ERR_WORKSPACE);
  EXPECT(spa2_bwd(fake, fake, fake, fake, odd, fake, (float*)fake, &ok, &full, 0.1f, fake, fake, fake, fake, big, 0),
         SPA2_ERR_ALIGN);
  EXPECT(spa2_bwd_delta(fake, 0, fake, &ok, fake, 8, 0), SPA2_ERR_WORKSPACE);
  EXPECT(spa2_bwd_dkdv(fake, fake, fake, fake, (float*)fake, &ok, &rows_only, 0.1f, fake, fake, fake, big, 0), SPA2_ERR_NULL);
  EXPECT(spa2_bwd_dq(fake, fake, fake, fake, (float*)fake, &ok, &full, -1.0f, fake, fake, big, 0), SPA2_ERR_RANGE);
  EXPECT(spa2_bwd_static(fake, fake, fake, fake, 0, fake, (float*)fake, 0, &full, 0.1f, fake, fake, fake, 0), SPA2_ERR_NULL);
  EXPECT(spa2_bwd_static(fake, fake, fake, fake, 0, fake, (float*)fake, &toolong, &full, 0.1f, fake, fake, fake, 0),
         SPA2_ERR_WORKSPACE);

  /* the backward pass that lists the columns itself: column lists may be missing, mask and row lists may not; a workspace that is a
     byte short, with the columns ranked by the launch of dQ (up to 4096 a head) and by one of their own */
#define BWD_ROWS(q, k, v, o, ores, d_o, lse, s, pat, sc, dq, dk, dv, ws, n) \
  spa2_bwd_rows(q, k, v, o, ores, d_o, (const float*)(lse), s, pat, sc, dq, dk, dv, ws, n, 0)
#define BWD_ROWS_OF(s, pat, sc, ws, n) BWD_ROWS(fake, fake, fake, fake, 0, fake, fake, s, pat, sc, fake, fake, fake, ws, n)
  {
    const spa2_shape edge = shape(1, 2, 64 * 4096, 64, 128, 64, 0), beyond = shape(1, 2, 64 * 4097, 64, 128, 64, 0);
    const spa2_shape* sizes[3] = {&ok, &edge, &beyond};
    const spa2_shape* bad[6] = {0, &d96, &bq64, &n0, &sn132, &huge};
    spa2_pattern no_mask = rows_only, no_cnt = rows_only, no_idx = rows_only;
    no_mask.mask = 0; no_cnt.row_cnt = 0; no_idx.row_idx = 0;
    for (int x = 0; x < 3; ++x) {
      const size_t need = spa2_bwd_rows_workspace_bytes(sizes[x]);
      if (need <= spa2_bwd_workspace_bytes(sizes[x])) { printf("bwd_rows size\n"); ++failures; }
      EXPECT(BWD_ROWS_OF(sizes[x], &rows_only, 0.1f, fake, need - 1), SPA2_ERR_WORKSPACE);
      EXPECT(BWD_ROWS_OF(sizes[x], &rows_only, 0.1f, 0, need), SPA2_ERR_WORKSPACE);
      EXPECT(BWD_ROWS_OF(sizes[x], &rows_only, 0.1f, odd, need), SPA2_ERR_ALIGN);
    }
    for (int x = 0; x < 6; ++x)
      if (spa2_bwd_rows_workspace_bytes(bad[x]) != 0) { printf("bwd_rows size of a bad shape\n"); ++failures; }
    EXPECT(BWD_ROWS_OF(&ok, 0, 0.1f, fake, big), SPA2_ERR_NULL);
    EXPECT(BWD_ROWS_OF(&ok, &none, 0.1f, fake, big), SPA2_ERR_NULL);
    EXPECT(BWD_ROWS_OF(&ok, &no_mask, 0.1f, fake, big), SPA2_ERR_NULL);
    EXPECT(BWD_ROWS_OF(&ok, &no_cnt, 0.1f, fake, big), SPA2_ERR_NULL);
    EXPECT(BWD_ROWS_OF(&ok, &no_idx, 0.1f, fake, big), SPA2_ERR_NULL);
    for (int x = 0; x < 10; ++x) {             /* each tensor missing, then misaligned (o_res may be missing, lse is fp32) */
      void* t[10];
      for (int y = 0; y < 10; ++y) t[y] = fake;
      t[x] = 0;
      if (x != 4)
        EXPECT(BWD_ROWS(t[0], t[1], t[2], t[3], t[4], t[5], t[6], &ok, &rows_only, 0.1f, t[7], t[8], t[9], fake, big), SPA2_ERR_NULL);
      t[x] = odd;
      if (x != 6)
        EXPECT(BWD_ROWS(t[0], t[1], t[2], t[3], t[4], t[5], t[6], &ok, &rows_only, 0.1f, t[7], t[8], t[9], fake, big), SPA2_ERR_ALIGN);
    }
    EXPECT(BWD_ROWS_OF(&ok, &rows_only, 0.0f, fake, big), SPA2_ERR_RANGE);
    EXPECT(BWD_ROWS_OF(&ok, &rows_only, -1.0f, fake, big), SPA2_ERR_RANGE);
    EXPECT(BWD_ROWS_OF(&ok, &rows_only, NAN, fake, big), SPA2_ERR_RANGE);
    EXPECT(BWD_ROWS_OF(&ok, &rows_only, INFINITY, fake, big), SPA2_ERR_RANGE);
    EXPECT(BWD_ROWS_OF(0, &rows_only, 0.1f, fake, big), SPA2_ERR_NULL);
    EXPECT(BWD_ROWS_OF(&d96, &rows_only, 0.1f, fake, big), SPA2_ERR_UNSUPPORTED);
    EXPECT(BWD_ROWS_OF(&bq64, &rows_only, 0.1f, fake, big), SPA2_ERR_UNSUPPORTED);
    EXPECT(BWD_ROWS_OF(&n0, &rows_only, 0.1f, fake, big), SPA2_ERR_SHAPE);
    EXPECT(BWD_ROWS_OF(&sn132, &rows_only, 0.1f, fake, big), SPA2_ERR_ALIGN);
    EXPECT(BWD_ROWS_OF(&wide, &rows_only, 0.1f, fake, big), SPA2_ERR_SHAPE);
    EXPECT(BWD_ROWS_OF(&many, &rows_only, 0.1f, fake, big), SPA2_ERR_SHAPE);
    EXPECT(BWD_ROWS_OF(&huge, &rows_only, 0.1f, fake, big), SPA2_ERR_SHAPE);
    EXPECT(BWD_ROWS_OF(&longrow, &rows_only, 0.1f, fake, big), SPA2_ERR_SHAPE);
  }

  EXPECT(spa2_error_terms(fake, fake, (float*)fake, (float*)fake, &ok, 0, fake, big, 0), SPA2_ERR_NULL);
  EXPECT(spa2_error_terms(fake, fake, (float*)fake, (float*)fake, &ok, (double*)fake, fake, 8, 0), SPA2_ERR_WORKSPACE);
  EXPECT(spa2_vd_loss(0, fake, 8, SPA2_DTYPE_BF16, 1.0, (double*)fake, fake, big, 0), SPA2_ERR_NULL);
  EXPECT(spa2_vd_loss(fake, fake, 0, SPA2_DTYPE_BF16, 1.0, (double*)fake, fake, big, 0), SPA2_ERR_SHAPE);
  EXPECT(spa2_vd_loss(fake, fake, 8, 2, 1.0, (double*)fake, fake, big, 0), SPA2_ERR_UNSUPPORTED);
  EXPECT(spa2_vd_loss(odd, fake, 8, SPA2_DTYPE_F32, 1.0, (double*)fake, fake, big, 0), SPA2_ERR_ALIGN);
  EXPECT(spa2_vd_loss(fake, fake, 8, SPA2_DTYPE_F32, INFINITY, (double*)fake, fake, big, 0), SPA2_ERR_RANGE);
  EXPECT(spa2_vd_loss(fake, fake, 8, SPA2_DTYPE_F32, 1.0, (double*)fake, fake, 64, 0), SPA2_ERR_WORKSPACE);
  EXPECT(spa2_vd_loss_grad(fake, fake, 8, SPA2_DTYPE_F32, 1.0, 0, 0, 0), SPA2_ERR_NULL);

  EXPECT(spa2_vd_loss_and_grad(0, fake, 8, 1.0, (double*)fake, fake, fake, big, 0), SPA2_ERR_NULL);
  EXPECT(spa2_vd_loss_and_grad(fake, fake, 8, 1.0, 0, fake, fake, big, 0), SPA2_ERR_NULL);
  EXPECT(spa2_vd_loss_and_grad(fake, fake, 8, 1.0, (double*)fake, 0, fake, big, 0), SPA2_ERR_NULL);
  EXPECT(spa2_vd_loss_and_grad(fake, fake, 0, 1.0, (double*)fake, fake, fake, big, 0), SPA2_ERR_SHAPE);
  EXPECT(spa2_vd_loss_and_grad(fake, odd, 8, 1.0, (double*)fake, fake, fake, big, 0), SPA2_ERR_ALIGN);
  EXPECT(spa2_vd_loss_and_grad(fake, fake, 8, 1.0, (double*)fake, odd, fake, big, 0), SPA2_ERR_ALIGN);
  EXPECT(spa2_vd_loss_and_grad(fake, fake, 8, 1.0, (double*)fake, fake, odd, big, 0), SPA2_ERR_ALIGN);
  EXPECT(spa2_vd_loss_and_grad(fake, fake, 8, -1.0, (double*)fake, fake, fake, big, 0), SPA2_ERR_RANGE);
  EXPECT(spa2_vd_loss_and_grad(fake, fake, 8, NAN, (double*)fake, fake, fake, big, 0), SPA2_ERR_RANGE);
  EXPECT(spa2_vd_loss_and_grad(fake, fake, 8, 5e-39, (double*)fake, fake, fake, big, 0), SPA2_ERR_RANGE);  /* 2w is subnormal */
  EXPECT(spa2_vd_loss_and_grad(fake, fake, 8, 1e300, (double*)fake, fake, fake, big, 0), SPA2_ERR_RANGE);
  EXPECT(spa2_vd_loss_and_grad(fake, fake, 8, 1.0, (double*)fake, fake, 0, big, 0), SPA2_ERR_WORKSPACE);
  EXPECT(spa2_vd_loss_and_grad(fake, fake, 8, 1.0, (double*)fake, fake, fake, spa2_vd_loss_workspace_bytes() - 1, 0),
         SPA2_ERR_WORKSPACE);
  EXPECT(spa2_vd_rescale(0, 8, 1.0, (double*)fake, 0), SPA2_ERR_NULL);
  EXPECT(spa2_vd_rescale(fake, 8, 1.0, 0, 0), SPA2_ERR_NULL);
  EXPECT(spa2_vd_rescale(fake, -1, 1.0, (double*)fake, 0), SPA2_ERR_SHAPE);
  EXPECT(spa2_vd_rescale(odd, 8, 1.0, (double*)fake, 0), SPA2_ERR_ALIGN);
  EXPECT(spa2_vd_rescale(fake, 8, 0.0, (double*)fake, 0), SPA2_ERR_RANGE);
  EXPECT(spa2_vd_rescale(fake, 8, 5e-39, (double*)fake, 0), SPA2_ERR_RANGE);

  /* pattern and forward pass in one call: what either refuses, and a workspace that is a byte short, on either side of the
     sizes that need no plan */
#define MASK_FWD(q, k, v, s, topk, p, sc, pat, o, ores, lse, ws, n) \
  spa2_mask_fwd(q, k, v, s, topk, p, sc, pat, o, ores, (float*)(lse), ws, n, 0)
  {
    const spa2_shape plan = shape(1, 17, 2048, 64, 128, 64, 0);
    const spa2_shape* sizes[2] = {&ok, &plan};
    for (int x = 0; x < 2; ++x) {
      const size_t need = spa2_mask_fwd_workspace_bytes(sizes[x]);
      if (need < spa2_fwd_workspace_bytes(sizes[x]) || need < spa2_mask_workspace_bytes(sizes[x])) { printf("mask_fwd size\n"); ++failures; }
      EXPECT(MASK_FWD(fake, fake, fake, sizes[x], 1, 0.5f, 0.1f, &full, fake, 0, fake, fake, need - 1), SPA2_ERR_WORKSPACE);
    }
    if (spa2_mask_fwd_workspace_bytes(0) != 0 || spa2_mask_fwd_workspace_bytes(&d96) != 0) { printf("mask_fwd size\n"); ++failures; }
  }
  EXPECT(MASK_FWD(fake, fake, fake, 0, 1, 0.5f, 0.1f, &full, fake, 0, fake, fake, big), SPA2_ERR_NULL);
  EXPECT(MASK_FWD(0, fake, fake, &ok, 1, 0.5f, 0.1f, &full, fake, 0, fake, fake, big), SPA2_ERR_NULL);
  EXPECT(MASK_FWD(fake, fake, 0, &ok, 1, 0.5f, 0.1f, &full, fake, 0, fake, fake, big), SPA2_ERR_NULL);
  EXPECT(MASK_FWD(fake, fake, fake, &ok, 1, 0.5f, 0.1f, 0, fake, 0, fake, fake, big), SPA2_ERR_NULL);
  EXPECT(MASK_FWD(fake, fake, fake, &ok, 1, 0.5f, 0.1f, &half, fake, 0, fake, fake, big), SPA2_ERR_NULL);
  EXPECT(MASK_FWD(fake, fake, fake, &ok, 1, 0.5f, 0.1f, &full, 0, 0, fake, fake, big), SPA2_ERR_NULL);
  EXPECT(MASK_FWD(fake, fake, fake, &ok, 1, 0.5f, 0.1f, &full, fake, 0, 0, fake, big), SPA2_ERR_NULL);
  EXPECT(MASK_FWD(odd, fake, fake, &ok, 1, 0.5f, 0.1f, &full, fake, 0, fake, fake, big), SPA2_ERR_ALIGN);
  EXPECT(MASK_FWD(fake, fake, odd, &ok, 1, 0.5f, 0.1f, &full, fake, 0, fake, fake, big), SPA2_ERR_ALIGN);
  EXPECT(MASK_FWD(fake, fake, fake, &ok, 1, 0.5f, 0.1f, &full, fake, odd, fake, fake, big), SPA2_ERR_ALIGN);
  EXPECT(MASK_FWD(fake, fake, fake, &ok, 1, 0.5f, 0.1f, &full, fake, 0, fake, odd, big), SPA2_ERR_ALIGN);
  EXPECT(MASK_FWD(fake, fake, fake, &ok, 1, 0.5f, 0.1f, &full, fake, 0, fake, 0, big), SPA2_ERR_WORKSPACE);
  EXPECT(MASK_FWD(fake, fake, fake, &ok, 6, 0.5f, 0.1f, &full, fake, 0, fake, fake, big), SPA2_ERR_RANGE);
  EXPECT(MASK_FWD(fake, fake, fake, &ok, 0, 0.0f, 0.1f, &full, fake, 0, fake, fake, big), SPA2_ERR_RANGE);
  EXPECT(MASK_FWD(fake, fake, fake, &ok, 1, NAN, 0.1f, &full, fake, 0, fake, fake, big), SPA2_ERR_RANGE);
  EXPECT(MASK_FWD(fake, fake, fake, &ok, 1, 0.5f, 0.0f, &full, fake, 0, fake, fake, big), SPA2_ERR_RANGE);
  EXPECT(MASK_FWD(fake, fake, fake, &d96, 1, 0.5f, 0.1f, &full, fake, 0, fake, fake, big), SPA2_ERR_UNSUPPORTED);
  EXPECT(MASK_FWD(fake, fake, fake, &longrow, 1, 0.5f, 0.1f, &full, fake, 0, fake, fake, big), SPA2_ERR_SHAPE);
  EXPECT(MASK_FWD(fake, fake, fake, &huge, 1, 0.5f, 0.1f, &full, fake, 0, fake, fake, big), SPA2_ERR_SHAPE);

  /* host helpers and size queries over their whole argument range */
  if (spa2_topk_blocks(0.2, 10) != 2 || spa2_topk_blocks(0.0, 10) != 0 || spa2_topk_blocks(5.0, 10) != 10 ||
      spa2_topk_blocks(NAN, 10) != 0 || spa2_topk_blocks(0.5, -3) != 0 || spa2_topk_blocks(1e300, 0x7fffffff) != 0x7fffffff) {
    printf("spa2_topk_blocks\n"); ++failures;
  }
  if (spa2_mask_workspace_bytes(&huge) != 0 || spa2_bwd_workspace_bytes(&d96) != 0 || spa2_mask_workspace_bytes(0) != 0 ||
      spa2_error_workspace_bytes(&n0) != 0 || spa2_mask_workspace_bytes(&ok) == 0 || spa2_bwd_workspace_bytes(&ok) == 0 ||
      spa2_fwd_workspace_bytes(&ok) == 0 || spa2_fwd_workspace_bytes(&d96) != 0 ||
      spa2_bwd_workspace_min_bytes(&ok) == 0 || spa2_bwd_workspace_min_bytes(&ok) > spa2_bwd_workspace_bytes(&ok)) {
    printf("workspace sizes\n"); ++failures;
  }
  for (int c = 1; c >= -9; --c)
    if (!spa2_strerror(c) || !spa2_strerror(c)[0]) { printf("strerror %d\n", c); ++failures; }
  printf(failures ? "FAILED %d\n" : "all rejected before launch\n", failures);
  return failures ? 1 : 0;
}
