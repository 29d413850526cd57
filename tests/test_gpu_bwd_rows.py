"""The backward pass that makes its own column lists against spa2_mask_columns and spa2_bwd: same bits."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2602_13515_amd as spa2
from paper_2602_13515_amd import workloads as wl

from gpu_util import Guarded, dev, dkdv_drawn, gpu_bwd, gpu_fwd, gpu_mask, plan_offsets

pytestmark = pytest.mark.gpu


# one block; a head of 64 and of 65 key blocks (edges of the listing and ranking workgroups), of 21 (blocks dealt in turn);
# 257 query blocks, listed 16, 32 and 64 columns a workgroup (9, 72 and 135 workgroups of 64); runs of query blocks longer than a
# register holds (15 heads of 257, 65 a thread; one of 2048, 128 a thread); 4096 and 4097 key blocks, on either side of what the
# dQ launch orders; 32,768 and 33,390 columns in all, on either side of what it lists in stretches; launches from a queue (at
# d = 64 32,768, 33,390 and 4,160 columns, at d = 128 4,100) and direct ones, in one round and in several
@pytest.mark.parametrize("B,H,N,d", [(1, 1, 40, 128), (2, 3, 4096, 64), (1, 2, 4100, 128), (4, 6, 1281, 128), (1, 1, 65600, 64),
                                     (1, 12, 11200, 64), (1, 1, 262144, 64), (1, 1, 262145, 64), (8, 64, 4096, 64),
                                     (6, 105, 3392, 64), (1, 41, 6400, 128), (1, 25, 3900, 128),
                                     (1, 1, 32832, 64), (1, 8, 32832, 64), (1, 15, 32832, 64), (1, 65, 4096, 64)])
@pytest.mark.parametrize("alike", [True, False])
def test_backward_from_the_mask_gives_the_bits_of_columns_and_backward(B, H, N, d, alike):
    w = wl.Workload("rows", B, H, N, d, 0.05, 0.3, "lowrank", True)
    q, k, v, do = (t.to(dev()) for t in wl.make_inputs(w, seed=2, **({"device": "cuda"} if B * H > 100 else {})))
    scale = d ** -0.5
    if not alike:                       # the first heads of the first sample select most of what the others select a few blocks of
        if N > 20000:
            pytest.skip("one size of head is enough")
        q[0, :max(1, H // 8)] *= 0.01
    pat, _ = gpu_mask(q, k, spa2.spa2_topk_blocks(0.05 if N < 200000 else 0.002, -(-N // 64)),
                      (0.3 if alike else 0.7) if N < 200000 else 0.0, scale, want_pbar=False)
    o, lse, o_res = gpu_fwd(q, k, v, pat, scale, residual=True)
    want = gpu_bwd(q, k, v, o, do, lse, pat, scale, o_res=o_res)
    lib, g, lay = spa2.binding._load(), Guarded(), spa2.binding._layout_of(q)
    need = int(lib.spa2_bwd_rows_workspace_bytes(lay.ref))
    ws = g.alloc((need,), torch.uint8, dev(), 0xA5)
    out = [g.alloc(q.shape, q.dtype, dev(), float("nan")) for _ in range(3)]
    rows = spa2.Pattern(pat.mask, pat.row_cnt, pat.row_idx, None, None, None, None)
    c = rows._c()
    ptr = lambda *ts: [t.data_ptr() for t in ts]
    call = lambda nbytes: lib.spa2_bwd_rows(*ptr(q, k, v, o, o_res, do, lse), lay.ref, ctypes.byref(c), scale, *ptr(*out),
                                            ws.data_ptr(), nbytes, spa2.binding._stream(q))
    assert call(need - 1) == -6
    print(f"case B={B} H={H} N={N} d={d}", flush=True)
    for _ in range(2):
        assert call(need) == 0
        torch.cuda.synchronize()
        g.check("spa2_bwd_rows")
        for name, x, y in zip(("dq", "dk", "dv"), out, want):
            assert torch.equal(x, y), name
    # what the plan of dK/dV says of the eighths of the columns, where they are launched in stretches, and how they are launched
    Tm, Tn = pat.mask.shape[2:]
    columns = B * H * Tn
    if Tm < 512 and columns <= 32768:
        cnt = pat.col_cnt.cpu().numpy().reshape(-1).astype(np.int64)
        eighth = np.bincount(np.minimum((np.arange(columns) * np.float32(8 / columns)).astype(int), 7), cnt, 8)
        even = 8 * eighth.max() <= cnt.sum() + cnt.sum() // 16
        at = plan_offsets(q)["dkdv"]
        assert int(ws[at:at + 12].view(torch.int32)[2]) == int(even)
        assert alike or B * H == 1 or not even
    resident = 1024 if d == 64 else 512
    if columns > 4 * resident:
        assert sum(dkdv_drawn(q, ws)) >= 2 * resident
