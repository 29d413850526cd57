"""Shared plumbing for the GPU parity tests: moves seeded inputs to the device, calls the
C ABI through the binding, and brings results back as float64 numpy arrays."""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2602_13515_amd as spa2
from oracle import spa2_oracle as orc

MAX_ABS = 2e-2    # tolerance on O, dQ, dK, dV fixed by the benchmark definition (bf16 outputs)
MEAN_ABS = 2e-3
LOWRANK_MAX_ABS = 5e-2   # dQ, dK on inputs with the rank-4 scale-2 component: derived in tests/test_tolerance_model.py
REL_L2 = 1.5e-2    # ||got - ref|| / ||ref|| per compared array; measured at most 7e-3 (dQ), 2e-3 (O)
PBAR_REL = 1e-5   # pooled-map scores: fp32 pooled means, fp64 dot products, fp32 softmax
CUT_EPS = 1e-5    # rows whose cumulative mass at the cut is this close to p may flip


def dev():
    return torch.device("cuda:0")


# ---- canaries: every output buffer of a call sits between two guard zones holding a sentinel pattern; after the
# call the zones must be untouched (an out-of-bounds write next to a buffer shows here, a NaN fill only shows
# elements that were never written)
GUARD_BYTES = 4096
_SENTINEL = 0xA5


class Guarded:
    def __init__(self):
        self.items = []

    def alloc(self, shape, dtype, device, fill):
        n = int(np.prod(shape))
        esz = torch.empty((), dtype=dtype).element_size()
        raw = torch.full((n * esz + 2 * GUARD_BYTES,), _SENTINEL, dtype=torch.uint8, device=device)
        body = raw[GUARD_BYTES:GUARD_BYTES + n * esz].view(dtype).view(shape)
        body.fill_(fill)
        self.items.append((raw, n * esz))
        return body

    def check(self, where=""):
        for raw, nbytes in self.items:
            lo, hi = raw[:GUARD_BYTES], raw[GUARD_BYTES + nbytes:]
            assert bool((lo == _SENTINEL).all()) and bool((hi == _SENTINEL).all()), \
                f"{where}: a kernel wrote outside an output buffer of {nbytes} bytes"


def guarded_pattern(g: Guarded, B, H, N, device, columns=True):
    Tm, Tn = -(-N // 128), -(-N // 64)
    i32 = torch.int32
    return spa2.Pattern(
        mask=g.alloc((B, H, Tm, Tn), torch.uint8, device, 7),
        row_cnt=g.alloc((B, H, Tm), i32, device, -1),
        row_idx=g.alloc((B, H, Tm, Tn), i32, device, -1),
        col_cnt=g.alloc((B, H, Tn), i32, device, -1) if columns else None,
        col_idx=g.alloc((B, H, Tn, Tm), i32, device, -1) if columns else None,
        col_order=g.alloc((B, H, Tn), i32, device, -1) if columns else None)


def f64(t: torch.Tensor) -> np.ndarray:
    return t.detach().to("cpu").double().numpy()


def pattern_from_mask(mask: np.ndarray, device) -> spa2.Pattern:
    """Index lists for a given 0/1 block mask [B,H,Tm,Tn] (test-side plumbing: a caller may
    hand the attention kernels any pattern)."""
    B, H, Tm, Tn = mask.shape
    row_cnt = mask.sum(-1).astype(np.int32)
    col_cnt = mask.sum(-2).astype(np.int32)
    row_idx = np.zeros((B, H, Tm, Tn), np.int32)
    col_idx = np.zeros((B, H, Tn, Tm), np.int32)
    for b in range(B):
        for h in range(H):
            for i in range(Tm):
                js = np.flatnonzero(mask[b, h, i])
                row_idx[b, h, i, :js.size] = js
            for j in range(Tn):
                is_ = np.flatnonzero(mask[b, h, :, j])
                col_idx[b, h, j, :is_.size] = is_
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(device)
    return spa2.Pattern(t(mask.astype(np.uint8)), t(row_cnt), t(row_idx), t(col_cnt), t(col_idx))


def gpu_mask(q, k, k_cnt, top_p, scale=None, want_pbar=True, columns=True):
    B, H, N, d = q.shape
    scale = 1.0 / math.sqrt(d) if scale is None else scale
    g = Guarded()
    pat = guarded_pattern(g, B, H, N, q.device, columns)     # poisoned, so that unwritten entries show
    Tm, Tn = pat.mask.shape[2:]
    pbar = g.alloc((B, H, Tm, Tn), torch.float32, q.device, float("nan")) if want_pbar else None
    ws = g.alloc((spa2.spa2_mask_workspace_bytes(q),), torch.uint8, q.device, 0)
    spa2.spa2_mask(q, k, k_cnt, top_p, scale, pat, pbar, ws)
    torch.cuda.synchronize()
    g.check("spa2_mask")
    return pat, pbar


# ---- what a call's split plans say (header of a plan: number of parts, list entries per part at most).  The forward
# workspace is one plan section, the backward workspace holds D, the section of the dQ kernel and that of the dK/dV one.
def _plan_section_bytes(units, list_max, slot_floats):
    up = lambda x: -(-x // 256) * 256
    per_unit = min(max(list_max // 2, 1), 16)
    pool = 8
    while pool < 2048 and pool < per_unit * units:
        pool *= 2
    return up(256 + up(units * 4) + up(pool * 16) + up(pool * 4) + pool * slot_floats * 4)


def plan_offsets(q):
    B, H, N, d = q.shape
    Tm, Tn = -(-N // spa2.BQ), -(-N // spa2.BKV)
    at = spa2.spa2_bwd_workspace_min_bytes(q)
    return {"fwd": 0, "dq": at, "dkdv": at + _plan_section_bytes(B * H * Tm, Tn, 256 * (d // 2))}


def plan_headers(q, ws, names=("dq", "dkdv")):
    """{name: (parts, entries per part)} of the plans in a forward (names = ("fwd",)) or backward workspace."""
    off = plan_offsets(q)
    return {n: tuple(ws[off[n]:off[n] + 8].view(torch.int32).tolist()) for n in names}


def dkdv_drawn(q, ws):
    """How many items each of the eight counters of the dK/dV queue has given out, in a backward workspace of full size that was
    zeros before the call: more than what the plan sets them to where the launch drew from the queue, just that where it was made
    for both ways and went the direct one, nothing where there is no queue."""
    B, H, N, d = q.shape
    Tm, Tn = -(-N // spa2.BQ), -(-N // spa2.BKV)
    units, per_unit, pool, up = B * H * Tn, min(max(Tm // 2, 1), 16), 8, lambda x: -(-x // 256) * 256
    while pool < 2048 and pool < per_unit * units:
        pool *= 2
    at = plan_offsets(q)["dkdv"] + 256 + up(units * 4) + up(pool * 16) + up(pool * 4) + (pool - 1) * 128 * d * 4
    return ws[at:at + 2048].view(torch.int32)[::64].tolist()


def check_plan(name, header, lengths):
    """The plan cut every list longer than its part length, and no other.  Returns the part length."""
    parts, S = header
    lengths = lengths.astype(np.int64)
    cut = lengths[lengths > S]
    print(f"{name}: parts of at most {S} entries; {cut.size} of {lengths.size} lists cut into {parts} parts", flush=True)
    assert parts == int((-(-cut // S)).sum()), (name, header)
    return S


def gpu_fwd(q, k, v, pat, scale=None, residual=False, split=True, plans=None):
    B, H, N, d = q.shape
    scale = 1.0 / math.sqrt(d) if scale is None else scale
    g = Guarded()
    o = g.alloc(q.shape, q.dtype, q.device, float("nan"))
    o_res = g.alloc(q.shape, q.dtype, q.device, float("nan")) if residual else None
    lse = g.alloc((B, H, N), torch.float32, q.device, float("nan"))
    # with the workspace, rows longer than the split length are walked by several workgroups
    ws = g.alloc((spa2.spa2_fwd_workspace_bytes(q),), torch.uint8, q.device, 0) if split else None
    spa2.spa2_fwd(q, k, v, pat, scale, o, lse, o_res, ws)
    torch.cuda.synchronize()
    g.check("spa2_fwd")
    if plans is not None:
        plans.update(plan_headers(q, ws, ("fwd",)))
    return (o, lse, o_res) if residual else (o, lse)


def gpu_bwd(q, k, v, o, do, lse, pat, scale=None, o_res=None, split=True, plans=None):
    d = q.shape[-1]
    scale = 1.0 / math.sqrt(d) if scale is None else scale
    g = Guarded()
    dq, dk, dv = (g.alloc(q.shape, q.dtype, q.device, float("nan")) for _ in range(3))
    nbytes = spa2.spa2_bwd_workspace_bytes(q) if split else spa2.spa2_bwd_workspace_min_bytes(q)
    ws = g.alloc((nbytes,), torch.uint8, q.device, 0)
    spa2.spa2_bwd(q, k, v, o, do, lse, pat, scale, dq, dk, dv, ws, o_res)
    torch.cuda.synchronize()
    g.check("spa2_bwd")
    if plans is not None:
        plans.update(plan_headers(q, ws))
        if split:
            plans["drawn"] = dkdv_drawn(q, ws)
    return dq, dk, dv


def check_pattern_consistency(pat: spa2.Pattern):
    """The three encodings of a pattern agree: counts, ascending lists, mask bits."""
    mask = pat.mask.cpu().numpy()
    assert set(np.unique(mask).tolist()) <= {0, 1}
    B, H, Tm, Tn = mask.shape
    row_cnt = pat.row_cnt.cpu().numpy(); row_idx = pat.row_idx.cpu().numpy()
    assert np.array_equal(row_cnt, mask.sum(-1))
    for b in range(B):
        for h in range(H):
            for i in range(Tm):
                assert np.array_equal(row_idx[b, h, i, :row_cnt[b, h, i]], np.flatnonzero(mask[b, h, i]))
    if pat.col_cnt is not None:
        col_cnt = pat.col_cnt.cpu().numpy(); col_idx = pat.col_idx.cpu().numpy()
        assert np.array_equal(col_cnt, mask.sum(-2))
        for b in range(B):
            for h in range(H):
                for j in range(Tn):
                    assert np.array_equal(col_idx[b, h, j, :col_cnt[b, h, j]], np.flatnonzero(mask[b, h, :, j]))
    if pat.col_order is not None:
        order = pat.col_order.cpu().numpy()
        assert np.array_equal(np.sort(order, axis=-1), np.broadcast_to(np.arange(Tn), order.shape)), \
            "col_order must be a permutation of the key blocks"
    return mask


def mask_protocol(mask_gpu: np.ndarray, pbar_gpu: np.ndarray, pbar_ref: np.ndarray, k_cnt: int, top_p: float):
    """Three-stage mask comparison for one head.  Returns a dict of counts.
    Stage 1: exported scores vs the fp64 pooled map (relative tolerance).
    Stage 2: the oracle's selection rule run on the exported fp32 scores must reproduce the
             GPU mask bit for bit, except rows whose cumulative mass at the cut is within
             CUT_EPS of p (counted).
    Stage 3: Hamming distance to the all-fp64 mask; every differing row must be explained by
             a near-threshold cut or by a swap of two scores closer than 4 fp32 ulps."""
    top_p = float(np.float32(top_p))
    diff = np.abs(pbar_gpu.astype(np.float64) - pbar_ref)
    normal = pbar_ref >= 1e-30            # below that, fp32 runs out of mantissa bits (denormals from 1.2e-38 down)
    stage1 = float((diff[normal] / pbar_ref[normal]).max())
    assert (diff[~normal] <= 1e-35).all()
    ref2 = orc.hybrid_mask(pbar_gpu.astype(np.float64), k_cnt, top_p)
    order, n_p, n, csum = orc.prefix_lengths(pbar_gpu.astype(np.float64), k_cnt, top_p)
    diff_rows = np.flatnonzero((ref2 != mask_gpu).any(axis=1))
    flips2, bad2 = 0, 0
    for i in diff_rows:
        # distance of the cumulative sums around the cut from p
        near = np.abs(csum[i] - top_p).min() <= CUT_EPS
        if near:
            flips2 += 1
        else:
            bad2 += 1
    ref3 = orc.hybrid_mask(pbar_ref, k_cnt, top_p)
    _, _, n3, csum3 = orc.prefix_lengths(pbar_ref, k_cnt, top_p)
    ham = int((ref3 != mask_gpu).sum())
    rows3 = np.flatnonzero((ref3 != mask_gpu).any(axis=1))
    near3 = swap3 = unexplained3 = 0
    for i in rows3:
        if np.abs(csum3[i] - top_p).min() <= CUT_EPS:
            near3 += 1
            continue
        d = np.flatnonzero(ref3[i] != mask_gpu[i])
        vals = pbar_ref[i, d]
        # all entries that changed sides sit within a few fp32 ulps of each other
        if (vals.max() - vals.min()) <= 4 * np.spacing(np.float32(vals.max())):
            swap3 += 1
        else:
            unexplained3 += 1
    return dict(stage1_max_rel=stage1, stage2_rows_differ=int(diff_rows.size), stage2_near_cut=flips2,
                stage2_unexplained=bad2, stage3_hamming=ham, stage3_near_cut=near3, stage3_ulp_swap=swap3,
                stage3_unexplained=unexplained3, rows=int(mask_gpu.shape[0]))


BF16_ULP_REL = 2.0 ** -7   # spacing of bf16 numbers relative to the value (worst case, mantissa 1.0)


def assert_close(name, got: np.ndarray, ref: np.ndarray, max_abs=MAX_ABS, mean_abs=MEAN_ABS, rel_l2=REL_L2):
    """The benchmark's bar, max-abs <= 2e-2 and mean-abs <= 2e-3, stated for values of order one.
    The path stores bf16 and feeds bf16 P / dS to the second products, so its error is relative to the
    magnitude of what is being summed: a row (one token) of dK whose entries reach 20 cannot be within
    2e-2 (bf16 numbers are 0.125 apart there).  For such rows the bar scales with the row: an element may
    deviate by one bf16 spacing of the largest magnitude in its row, and the mean bar becomes 2^-8 of the mean
    magnitude.  Returns (max-abs, mean-abs, number of elements above the plain 2e-2) so callers can print
    how often the scaled bar was needed."""
    assert np.isfinite(got).all(), f"{name}: non-finite values in the GPU result"
    err = np.abs(got - ref)
    rowmax = np.abs(ref).max(axis=-1, keepdims=True)
    tol = np.maximum(max_abs, BF16_ULP_REL * rowmax)
    worst = int(np.argmax(err - tol))
    assert (err <= tol).all(), (f"{name}: |err| {err.flat[worst]:.4g} at |ref| {abs(ref.flat[worst]):.4g} "
                                f"exceeds max(2e-2, 2^-7 * row max); max-abs {err.max():.4g}")
    mean_bar = max(mean_abs, 2.0 ** -8 * float(np.abs(ref).mean()))   # rounding to bf16 alone costs about 2^-9.5 * mean|x|
    assert err.mean() <= mean_bar, f"{name}: mean-abs {err.mean():.4g} > {mean_bar:.4g}"
    # The absolute bar says little where the values themselves are small (long rows of near-uniform weights give
    # |O| of a few 1e-3), so the error is also bounded relative to the result: two bf16 roundings (P or dS, then
    # the stored output) give a relative L2 error of about 2e-3; dQ reaches 7e-3 through the cancellation in
    # dP - D.  A dropped tile, term or factor is ten times the bar or more.
    rel = float(np.linalg.norm(err) / max(np.linalg.norm(ref), 1e-300))
    assert rel <= rel_l2, f"{name}: relative L2 error {rel:.3g} > {rel_l2:.3g}"
    return float(err.max()), float(err.mean()), int((err > max_abs).sum())
