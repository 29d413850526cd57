"""Lists around the part length of the split plan: one entry, exactly one part, one entry more, last parts of one entry,
the whole range; with the full workspace, with ones whose pool (of the forward and the dQ kernel, of the dK/dV kernel)
is too small for the first choice of part length, and with none.  Each against the fp64 oracle, twice for the same
bits."""
import math

import numpy as np
import pytest
import torch

import paper_2602_13515_amd as spa2
from oracle import spa2_oracle as orc
from paper_2602_13515_amd import workloads as wl

from gpu_util import assert_close, check_plan, dev, f64, pattern_from_mask, plan_headers, plan_offsets

pytestmark = pytest.mark.gpu


def _mask(H, Tm, Tn):
    """Row i of head h keeps lengths[(i + h) % len] blocks spread over the row; block 0 in every row (one long column)."""
    lengths = [1, 2, 7, 8, 9, 15, 16, 17, 25, Tn]
    m = np.zeros((1, H, Tm, Tn), np.uint8)
    rng = np.random.default_rng(3)
    for h in range(H):
        for i in range(Tm):
            n = min(lengths[(i + h) % len(lengths)], Tn)
            m[0, h, i, 0] = 1
            m[0, h, i, 1 + rng.permutation(Tn - 1)[:n - 1]] = 1
    return m


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("N", [2500, 40])
@pytest.mark.parametrize("space", ["full", "small", "columns", "none"])
def test_part_edges(d, N, space):
    w = wl.Workload("parts", 1, 2, N, d, 0.1, 0.5, "gaussian", True)
    print(f"case d={d} N={N} workspace={space}", flush=True)
    q, k, v, do = wl.make_inputs(w, seed=11)
    mask = _mask(w.H, w.Tm, w.Tn)
    qd, kd, vd, dod = (t.to(dev()) for t in (q, k, v, do))
    pat = pattern_from_mask(mask, dev())
    nf, nb, nmin = (f(qd) for f in (spa2.spa2_fwd_workspace_bytes, spa2.spa2_bwd_workspace_bytes, spa2.spa2_bwd_workspace_min_bytes))
    dkdv_at = plan_offsets(qd)["dkdv"]
    if space == "small":        # room for a few slots only: the plans have to take longer parts (none for the columns)
        nf, nb = nf // 8, nmin + (nb - nmin) // 32
    elif space == "columns":    # the same for the columns alone
        nb = dkdv_at + (nb - dkdv_at) // 16
    elif space == "none":
        nf, nb = 0, nmin
    runs = []
    for _ in range(2):
        ws_f = torch.full((nf,), 0xA5, dtype=torch.uint8, device=dev()) if nf else None
        ws_b = torch.full((nb,), 0xA5, dtype=torch.uint8, device=dev())
        o, o_res, dq, dk, dv = (torch.full_like(qd, float("nan")) for _ in range(5))
        lse = torch.full((1, w.H, N), float("nan"), device=dev())
        spa2.spa2_fwd(qd, kd, vd, pat, 1 / math.sqrt(d), o, lse, o_res, ws_f)
        spa2.spa2_bwd(qd, kd, vd, o, dod, lse, pat, 1 / math.sqrt(d), dq, dk, dv, ws_b, o_res)
        torch.cuda.synchronize()
        if space == "full" or (space != "none" and N > 40):      # (40 tokens: nothing to cut, and no room for small plans)
            plans = plan_headers(qd, ws_b, ("dq",) if space == "small" else ("dq", "dkdv")) | plan_headers(qd, ws_f, ("fwd",))
            for name, header in plans.items():
                lengths = mask.sum(-2 if name == "dkdv" else -1)
                S = check_plan(name, header, lengths)
                assert N == 40 or lengths.max() > S, f"{name}: the case must cut some lists"
                if N > 40:      # the part length that the rule asks for on this pattern, longer where the pool is small
                    small = space == "small" or (space == "columns" and name == "dkdv")
                    first = {"fwd": 8, "dq": 8, "dkdv": 4}[name]
                    assert S > first if small else S == first, (name, header)
        runs.append((o, lse, o_res, dq, dk, dv))
        # the stage calls make their own plans: same bits as the composite call
        dq2, dk2, dv2 = (torch.full_like(qd, float("nan")) for _ in range(3))
        spa2.spa2_bwd_delta(o, dod, ws_b, o_res)
        spa2.spa2_bwd_dkdv(qd, kd, vd, dod, lse, pat, 1 / math.sqrt(d), dk2, dv2, ws_b)
        spa2.spa2_bwd_dq(qd, kd, vd, dod, lse, pat, 1 / math.sqrt(d), dq2, ws_b)
        torch.cuda.synchronize()
        for a, b in zip((dq, dk, dv), (dq2, dk2, dv2)):
            assert torch.equal(a, b)
    for a, b in zip(*runs):
        assert torch.equal(a, b), "results must not depend on the order in which parts finish"
    o, lse, o_res, dq, dk, dv = runs[0]
    r_dq, r_dk, r_dv, r_o, r_lse = orc.attention_bwd_bh(f64(q), f64(k), f64(v), mask, f64(do))
    assert_close("O", f64(o), r_o)
    assert np.abs(f64(lse) - r_lse).max() <= 2e-3
    assert_close("dQ", f64(dq), r_dq)
    assert_close("dK", f64(dk), r_dk)
    assert_close("dV", f64(dv), r_dv)


@pytest.mark.parametrize("rows", [8, 17, 25, 32, 33, 40, 59])
def test_every_row_is_launched_once(rows):
    """Rows per XCD (rows / 8, rounded up) around the groups of four that the launch order rotates: one block per row,
    so that every row's result is its own and a row that is left out or taken for another one shows."""
    N, H, d = 128 * rows - 5, 3, 64
    w = wl.Workload("order", 1, H, N, d, 0.1, 0.5, "gaussian", True)
    print(f"case rows={rows}", flush=True)
    q, k, v, do = (t.to(dev()) for t in wl.make_inputs(w, seed=rows))
    mask = np.zeros((1, H, w.Tm, w.Tn), np.uint8)
    for h in range(H):
        for i in range(w.Tm):
            mask[0, h, i, (7 * i + h) % w.Tn] = 1
    pat = pattern_from_mask(mask, dev())
    o, o_res, dq, dk, dv = (torch.full_like(q, float("nan")) for _ in range(5))
    lse = torch.full((1, H, N), float("nan"), device=dev())
    ws = torch.empty(spa2.spa2_bwd_workspace_bytes(q), dtype=torch.uint8, device=dev())
    spa2.spa2_fwd(q, k, v, pat, 1 / math.sqrt(d), o, lse, o_res)
    spa2.spa2_bwd(q, k, v, o, do, lse, pat, 1 / math.sqrt(d), dq, dk, dv, ws, o_res)
    torch.cuda.synchronize()
    r_dq, r_dk, r_dv, r_o, r_lse = orc.attention_bwd_bh(f64(q), f64(k), f64(v), mask, f64(do))
    assert np.abs(f64(lse) - r_lse).max() <= 2e-3
    for name, got, ref in (("O", o, r_o), ("dQ", dq, r_dq), ("dK", dk, r_dk), ("dV", dv, r_dv)):
        assert_close(name, f64(got), ref)


@pytest.mark.parametrize("rows,cols", [(1, 1), (1, 9), (3, 63), (2, 64), (5, 65), (2, 511), (3, 513), (1, 2049), (2, 8192)])
def test_column_order_is_longest_first_dealt_to_the_xcds(rows, cols):
    """col_order against a host sort, at the edges of the workgroups (64 columns) and of the instantiated widths."""
    B, H, N = 1, 2, 64 * cols
    like = torch.empty((B, H, N, 64), dtype=torch.bfloat16, device=dev())
    pat = spa2.alloc_pattern(B, H, N, dev())
    Tm, Tn = pat.mask.shape[-2:]
    print(f"case Tm={Tm} Tn={Tn}", flush=True)
    rng = np.random.default_rng(cols)
    mask = (rng.random((B, H, Tm, Tn)) < rng.random(Tn) ** rows).astype(np.uint8)
    pat.mask.copy_(torch.from_numpy(mask))
    spa2.spa2_mask_columns(like, pat)
    torch.cuda.synchronize()
    cnt = mask.sum(axis=2)
    assert np.array_equal(pat.col_cnt.cpu().numpy(), cnt)
    chunk = -(-Tn // 8)
    dealt = [x * chunk + s for s in range(chunk) for x in range(8) if s < min(max(Tn - x * chunk, 0), chunk)]
    for h in range(H):
        want = np.empty(Tn, np.int64)
        want[dealt] = np.argsort(-cnt[0, h].astype(np.int64), kind="stable")
        assert np.array_equal(pat.col_order[0, h].cpu().numpy(), want)
