"""dK/dV launches whose workgroups draw their columns from a queue against the direct launch of the same columns."""

import numpy as np
import pytest
import torch

import paper_2602_13515_amd as spa2
from paper_2602_13515_amd import workloads as wl

from gpu_util import check_plan, dev, dkdv_drawn, gpu_bwd, gpu_fwd, pattern_from_mask, plan_headers, plan_offsets

pytestmark = pytest.mark.gpu

# columns a launch takes directly: 2,048 at d = 128, where 512 workgroups run at a time, 4,096 at d = 64, where 1,024 do
DIRECT = {128: 2048, 64: 4096}


def queued(plans, d):
    """Whether the dK/dV launch drew its items: every workgroup that stays draws at least one beyond its first."""
    resident = DIRECT[d] // 4
    assert all(n == 0 for n in plans["drawn"]) or all(n >= resident // 8 for n in plans["drawn"])
    return sum(plans["drawn"]) >= 2 * resident


# on either side of the line; ragged and full last blocks; columns of 0 to 4 entries, which no plan cuts, so that both ways add the
# same products in the same order
@pytest.mark.parametrize("B,H,N,d", [(2, 64, 1000, 128), (1, 683, 190, 64), (2, 40, 1700, 128), (1, 129, 1024, 64),
                                     (2, 128, 1000, 64), (1, 1366, 190, 64), (1, 257, 1024, 64)])
def test_queue_gives_the_bits_of_the_direct_launch(B, H, N, d):
    w = wl.Workload("queue", B, H, N, d, 0.1, 0.5, "gaussian", True)
    q, k, v, do = (t.to(dev()) for t in wl.make_inputs(w, seed=5))
    Tm, Tn = -(-N // 128), -(-N // 64)
    rng = np.random.default_rng(7)
    mask = np.zeros((B, H, Tm, Tn), dtype=np.uint8)
    for _ in range(4):                                  # every row and most columns get one entry a round
        cols = rng.integers(0, Tn, size=(B, H, Tm))
        np.put_along_axis(mask, cols[..., None], 1, axis=-1)
    keep = np.cumsum(mask, axis=2) <= 4                 # at most four entries a column
    mask *= keep.astype(np.uint8)
    pat = pattern_from_mask(mask, dev())
    print(f"case B={B} H={H} N={N} d={d}", flush=True)
    o, lse, o_res = gpu_fwd(q, k, v, pat, residual=True)
    plans = {}
    first = gpu_bwd(q, k, v, o, do, lse, pat, o_res=o_res, plans=plans)
    assert queued(plans, d) == (B * H * Tn > DIRECT[d])
    direct = gpu_bwd(q, k, v, o, do, lse, pat, o_res=o_res, split=False)
    again = gpu_bwd(q, k, v, o, do, lse, pat, o_res=o_res)
    for name, x, y, z in zip(("dq", "dk", "dv"), first, direct, again):
        assert torch.equal(x, y), name
        assert torch.equal(x, z), name


# Columns of full length at d = 64: drawn where the last round of the direct launch would be up to three quarters full (1,025 to
# 1,792 columns of the first two rounds), from 16 query blocks and from 15/16 of all tiles on (one more is missing in the last
# case).  Two parts of every column would be more than the plan has room for: nothing is cut.
@pytest.mark.parametrize("H,N,d,missing,draws", [(48, 2048, 64, 0, True), (33, 2000, 64, 0, True), (56, 2048, 64, 0, True), (80, 2048, 64, 0, True),
                                                 (32, 2048, 64, 0, False), (57, 2048, 64, 0, False), (64, 2048, 64, 0, False),
                                                 (52, 1900, 64, 0, False), (48, 2048, 128, 0, False), (48, 2048, 64, 1536, True),
                                                 (48, 2048, 64, 1537, False)])
def test_full_columns_are_drawn_where_the_last_round_is_short(H, N, d, missing, draws):
    w = wl.Workload("queue", 1, H, N, d, 0.1, 0.5, "gaussian", True)
    q, k, v, do = (t.to(dev()) for t in wl.make_inputs(w, seed=6))
    Tm, Tn = -(-N // 128), -(-N // 64)
    mask = np.ones((1, H, Tm, Tn), dtype=np.uint8)
    mask.reshape(-1)[np.random.default_rng(3).permutation(mask.size)[:missing]] = 0
    pat = pattern_from_mask(mask, dev())
    print(f"case H={H} N={N} d={d} missing={missing}", flush=True)
    o, lse, o_res = gpu_fwd(q, k, v, pat, residual=True)
    plans = {}
    got = gpu_bwd(q, k, v, o, do, lse, pat, o_res=o_res, plans=plans)
    assert queued(plans, d) == draws
    want = gpu_bwd(q, k, v, o, do, lse, pat, o_res=o_res, split=False)
    x = [t.detach().clone().requires_grad_() for t in (q, k, v)]
    other = torch.autograd.grad(spa2.sparge_attn2(*x, 1.0, 0.0), x, do) if not missing else got      # (columns in stretches)
    for name, a, b, c in zip(("dk", "dv"), got[1:], want[1:], other[1:]):       # (rows of dQ are cut with a workspace)
        assert torch.equal(a, b), name
        assert torch.equal(a, c), name
    assert torch.equal(got[0], other[0])
    # the stage call, whose plan is a launch of its own, with room for a fifth of the parts
    at, full = plan_offsets(q)["dkdv"], spa2.spa2_bwd_workspace_bytes(q)
    ws = torch.zeros(at + (full - at) // 5, dtype=torch.uint8, device=dev())
    spa2.spa2_bwd_delta(o, do, ws, o_res)
    dk, dv = torch.full_like(q, float("nan")), torch.full_like(q, float("nan"))
    spa2.spa2_bwd_dkdv(q, k, v, do, lse, pat, d ** -0.5, dk, dv, ws)
    assert torch.equal(dk, want[1]) and torch.equal(dv, want[2])


def _cut_pattern(B, H, N, seed, every):
    """Most columns of two entries or so, a fifth of those of every fourth (eighth) head of all row blocks: these a plan cuts.
    Their launch order by the library."""
    Tm, Tn = -(-N // 128), -(-N // 64)
    rng = np.random.default_rng(seed)
    mask = np.zeros((B, H, Tm, Tn), dtype=np.uint8)
    for _ in range(4):
        np.put_along_axis(mask, rng.integers(0, Tn, size=(B, H, Tm))[..., None], 1, axis=-1)
    mask[:, ::every, :, rng.permutation(Tn)[:Tn // 5]] = 1
    pat = pattern_from_mask(mask, dev())
    order = spa2.alloc_pattern(B, H, N, dev())
    order.mask.copy_(pat.mask)
    spa2.spa2_mask_columns(torch.empty((B, H, N, 64), dtype=torch.bfloat16, device=dev()), order)
    return mask, pat, order.col_order


# heads of 55 columns and of 28 (dealt in turn); full workspace, and one whose pool is too small for the first choice of
# parts in the first case (110 columns of three parts, 255 slots); at d = 64 a direct launch of cut columns as well
@pytest.mark.parametrize("H,N,d,every", [(40, 3500, 128, 4), (75, 1790, 64, 4), (150, 1790, 64, 8)])
@pytest.mark.parametrize("space", ["full", "small"])
def test_queue_with_cut_columns(H, N, d, every, space):
    """Parts and whole columns from one queue: every column against the direct launch that cuts nothing, and the same bits with
    and without a launch order and from run to run."""
    w = wl.Workload("queue", 1, H, N, d, 0.1, 0.5, "gaussian", True)
    print(f"case H={H} N={N} d={d} {space}", flush=True)
    q, k, v, do = (t.to(dev()) for t in wl.make_inputs(w, seed=5))
    mask, pat, order = _cut_pattern(1, H, N, 7, every)
    o, lse, o_res = gpu_fwd(q, k, v, pat, residual=True)
    direct = gpu_bwd(q, k, v, o, do, lse, pat, o_res=o_res, split=False)
    at, full = plan_offsets(q)["dkdv"], spa2.spa2_bwd_workspace_bytes(q)
    nbytes = full if space == "full" else at + (full - at) // 5
    runs = []
    for col_order in (None, order, order):
        pat.col_order = col_order
        ws = torch.full((nbytes,), 0xA5, dtype=torch.uint8, device=dev())
        if space == "full":
            ws.zero_()
        out = tuple(torch.full_like(q, float("nan")) for _ in range(3))
        spa2.spa2_bwd(q, k, v, o, do, lse, pat, d ** -0.5, *out, ws, o_res)
        torch.cuda.synchronize()
        header = plan_headers(q, ws, ("dkdv",))["dkdv"]
        S = check_plan("dkdv", header, mask.sum(-2))
        # (the last slot holds the queue's counters)
        pool = 2048 if space == "full" else 256
        assert 0 < header[0] <= pool - 1 and mask.sum(-2).max() > S, (header, pool)
        if space == "full":
            assert queued({"drawn": dkdv_drawn(q, ws)}, d) == (H * mask.shape[-1] > DIRECT[d])
        runs.append(out)
    for out in runs[1:]:
        assert all(torch.equal(a, b) for a, b in zip(runs[0], out))
    # The products are the same, the fp32 sums of up to 3,584 of them run in another order: far below 2^-12 of a row's largest
    # value; then one rounding to bf16, up to a spacing apart (2^-7 of the value).
    for name, x, y in zip(("dq", "dk", "dv"), runs[0], direct):
        x, y = x.float(), y.float()
        bar = 2.0 ** -7 * torch.maximum(x.abs(), y.abs()) + 2.0 ** -12 * y.abs().amax(-1, keepdim=True)
        assert bool(((x - y).abs() <= bar).all()), name


# one, three and nine columns a head: no XCD is left without
@pytest.mark.parametrize("H,N,d", [(2100, 60, 64), (700, 190, 128), (240, 567, 64), (4200, 60, 64), (480, 567, 64)])
def test_queue_over_heads_of_a_few_columns(H, N, d):
    g = torch.Generator().manual_seed(2)
    q, k, v, do = (torch.randn((1, H, N, d), generator=g).bfloat16().to(dev()) for _ in range(4))
    pat = spa2.alloc_pattern(1, H, N, dev())
    spa2.spa2_pattern_full(q, pat)
    o, lse, o_res = gpu_fwd(q, k, v, pat, residual=True)
    plans = {}
    got = gpu_bwd(q, k, v, o, do, lse, pat, o_res=o_res, plans=plans)
    assert queued(plans, d) == (H * -(-N // 64) > DIRECT[d])
    direct = gpu_bwd(q, k, v, o, do, lse, pat, o_res=o_res, split=False)
    for name, x, y in zip(("dq", "dk", "dv"), got, direct):       # (five entries a column at most: nothing is cut)
        assert torch.equal(x, y), name
