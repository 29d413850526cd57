"""The selection kernels at the edges of their ranges: row widths and launch sizes on either side of the rules that choose
between four and sixteen rows per workgroup and between four and eight waves for the latter, and the sixteen-row
kernel's last row group."""
import numpy as np
import pytest

import paper_2602_13515_amd as spa2
from oracle import spa2_oracle as orc
from paper_2602_13515_amd import workloads as wl

from gpu_util import dev, f64, gpu_mask, mask_protocol

pytestmark = pytest.mark.gpu

CASES = [                                   # H, N, d, kind
    (2, 64 * 2, 64, "gaussian"),            # one row of two blocks: sixteen-row groups of one row
    (2, 64 * 128, 128, "lowrank"),          # the widest row that takes sixteen rows whatever the launch
    (2, 64 * 129 - 3, 64, "lowrank"),       # one block more, few workgroups: four rows per workgroup
    (16, 64 * 256, 64, "stress"),           # 128 groups of sixteen rows
    (15, 64 * 256, 128, "lowrank"),         # 120 of them
    (15, 64 * 257 - 9, 64, "lowrank"),      # 135 groups, the last of one row
    (3, 64 * 1537 - 1, 128, "lowrank"),
    (2, 64 * 2048 - 5, 64, "lowrank"),
    (1, 64 * 2048, 128, "stress"),          # widest row of the sixteen-row kernel, too few workgroups for it
    (2, 64 * 2049 - 64, 64, "gaussian"),    # 2048 blocks
    (2, 64 * 2049, 64, "lowrank"),          # 2049: four rows per workgroup
    # launches of 1024 groups of sixteen rows and more: four waves up to 1536 (d = 64) and 1280 (d = 128) blocks a row
    (1023, 64 * 20, 64, "gaussian"),        # one group short
    (1024, 64 * 20 - 7, 128, "lowrank"),
    (32, 64 * 1025 - 3, 64, "lowrank"),     # 1056 groups, the last of one row
    (26, 64 * 1280, 64, "stress"),          # the 1280-wide instantiation filled
    (25, 64 * 1281 - 60, 64, "lowrank"),    # 1025 groups; the widest four-wave instantiation, and its last row
    (22, 64 * 1536, 64, "lowrank"),
    (22, 64 * 1537, 64, "lowrank"),         # eight waves
    (26, 64 * 1280 - 1, 128, "lowrank"),    # d = 128: the widest row of the four-wave workgroups
    (25, 64 * 1281, 128, "stress"),         # eight waves
]


@pytest.mark.parametrize("H,N,d,kind", CASES, ids=[f"h{c[0]}-n{c[1]}-d{c[2]}-{c[3]}" for c in CASES])
def test_selection_at_the_edges(H, N, d, kind):
    print(f"case H={H} N={N} d={d} {kind}", flush=True)
    w = wl.Workload("edge", 1, H, N, d, 0.05, 0.7, kind, False)
    q, k, _, _ = wl.make_inputs(w, seed=6, need_do=False, device="cpu" if H <= 16 else dev())     # (the large ones: drawn there)
    k_cnt = spa2.spa2_topk_blocks(w.k_frac, w.Tn)
    pat, pbar = gpu_mask(q.to(dev()), k.to(dev()), k_cnt, w.top_p, columns=False)
    mask, cnt, idx = (t.cpu().numpy() for t in (pat.mask, pat.row_cnt, pat.row_idx))
    assert np.array_equal(cnt, mask.sum(-1))
    for h in sorted({0, H - 1}):
        for i in range(w.Tm):
            assert np.array_equal(idx[0, h, i, :cnt[0, h, i]], np.flatnonzero(mask[0, h, i]))
        r = mask_protocol(mask[0, h], pbar[0, h].cpu().numpy(), orc.pooled_map(f64(q[0, h]), f64(k[0, h])), k_cnt, w.top_p)
        assert r["stage1_max_rel"] <= 1e-5 and r["stage2_unexplained"] == 0 and r["stage3_unexplained"] == 0, r
