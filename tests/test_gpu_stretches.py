"""The order in which rows are launched (an eighth of all rows for each XCD, or of every head) changes no result."""
import numpy as np
import pytest
import torch

import paper_2602_13515_amd as spa2
from paper_2602_13515_amd import workloads as wl

from gpu_util import dev, gpu_bwd, gpu_fwd, pattern_from_mask, plan_offsets

pytestmark = pytest.mark.gpu


# fewer rows than XCDs, rows that no eight divide, heads of one row and of 33, 511 and 512 rows on either side of the rule
@pytest.mark.parametrize("H,N,d", [(1, 100, 64), (3, 200, 128), (50, 128, 64), (9, 4200, 128), (21, 1900, 64), (1, 511 * 128, 64),
                                   (1, 512 * 128, 64)])
@pytest.mark.parametrize("alike", [True, False])
def test_rows_in_stretches_and_by_heads(H, N, d, alike):
    w = wl.Workload("stretch", 1, H, N, d, 0.1, 0.5, "gaussian", True)
    q, k, v, do = (t.to(dev()) for t in wl.make_inputs(w, seed=5))
    Tm, Tn = -(-N // 128), -(-N // 64)
    rng = np.random.default_rng(7)
    mask = np.zeros((1, H, Tm, Tn), dtype=np.uint8)
    for r in range(4):                                  # up to four entries a row, one in most heads if these are not alike:
        cols = rng.integers(0, Tn, size=(1, H, Tm))     # no list of a row is cut
        some = np.ones((1, H, Tm, 1), dtype=np.uint8) if alike or r == 0 else (np.arange(H) < max(1, H // 6))[None, :, None, None]
        np.put_along_axis(mask, cols[..., None], np.maximum(np.take_along_axis(mask, cols[..., None], -1), some), axis=-1)
    pat = pattern_from_mask(mask, dev())
    print(f"case H={H} N={N} d={d} alike={alike}", flush=True)
    want = gpu_fwd(q, k, v, pat, residual=True, split=False)          # without a workspace: by heads
    got = gpu_fwd(q, k, v, pat, residual=True)
    for x, y in zip(want, got):
        assert torch.equal(x, y)
    o, lse, o_res = want
    assert torch.equal(gpu_bwd(q, k, v, o, do, lse, pat, o_res=o_res, split=False)[0], gpu_bwd(q, k, v, o, do, lse, pat, o_res=o_res)[0])
    # what the plan says of the eighths
    ws = torch.zeros(spa2.spa2_fwd_workspace_bytes(q), dtype=torch.uint8, device=dev())
    spa2.spa2_fwd(q, k, v, pat, d ** -0.5, torch.empty_like(q), torch.empty((1, H, N), device=dev()), None, ws)
    cnt = mask.sum(-1).reshape(-1).astype(np.int64)
    eighth = np.bincount(np.minimum((np.arange(cnt.size) * np.float32(8 / cnt.size)).astype(int), 7), cnt, 8)
    even = 8 * eighth.max() <= cnt.sum() + cnt.sum() // 16
    assert int(ws[:12].view(torch.int32)[2]) == int(even)
    if H >= 21 and N > 128:
        assert bool(even) == alike


# heads of 511 and 512 rows, on either side of the rule: the eighths are summed only where somebody reads what comes of it
@pytest.mark.parametrize("Tm", [511, 512])
def test_plan_sums_the_eighths_only_where_they_are_read(Tm):
    N = 128 * Tm
    mask = np.zeros((1, 2, Tm, 2 * Tm), dtype=np.uint8)
    mask[..., 0] = 1
    mask[0, 0, :, :8] = 1                               # the first head has eight times the entries of the second
    pat = pattern_from_mask(mask, dev())
    q = torch.zeros((1, 2, N, 64), dtype=torch.bfloat16, device=dev())
    ws = torch.zeros(spa2.spa2_fwd_workspace_bytes(q), dtype=torch.uint8, device=dev())
    spa2.spa2_fwd(q, q, q, pat, 0.125, torch.empty_like(q), torch.empty((1, 2, N), device=dev()), None, ws)
    assert int(ws[:12].view(torch.int32)[2]) == (0 if Tm < 512 else 1)
