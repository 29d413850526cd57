"""The selection kernel for rows of up to 64 blocks at the edges of its column tiles and row groups."""
import numpy as np
import pytest

import paper_2602_13515_amd as spa2
from oracle import spa2_oracle as orc
from paper_2602_13515_amd import workloads as wl

from gpu_util import dev, f64, gpu_mask, mask_protocol

pytestmark = pytest.mark.gpu


# 1, 2, 16, 17, 63, 64 blocks a row and 65 (the next kernel); one row, sixteen and seventeen rows a head
@pytest.mark.parametrize("N", [1, 65, 1024, 1025, 2048, 2049, 64 * 63 - 5, 64 * 64, 64 * 64 + 1])
@pytest.mark.parametrize("d,kind,k_frac,top_p", [(64, "lowrank", 0.1, 0.7), (128, "stress", 0.0, 0.9), (128, "gaussian", 0.3, 0.0)])
def test_short_rows(N, d, kind, k_frac, top_p):
    w = wl.Workload("small", 1, 3, N, d, k_frac, top_p, kind, False)
    q, k, _, _ = wl.make_inputs(w, seed=8, need_do=False)
    k_cnt = spa2.spa2_topk_blocks(k_frac, w.Tn)
    pat, pbar = gpu_mask(q.to(dev()), k.to(dev()), k_cnt, top_p, columns=False)
    mask, cnt, idx = (t.cpu().numpy() for t in (pat.mask, pat.row_cnt, pat.row_idx))
    assert np.array_equal(cnt, mask.sum(-1))
    for h in range(3):
        for i in range(w.Tm):
            assert np.array_equal(idx[0, h, i, :cnt[0, h, i]], np.flatnonzero(mask[0, h, i]))
        r = mask_protocol(mask[0, h], pbar[0, h].cpu().numpy(), orc.pooled_map(f64(q[0, h]), f64(k[0, h])), k_cnt, top_p)
        assert r["stage1_max_rel"] <= 1e-5 and r["stage2_unexplained"] == 0 and r["stage3_unexplained"] == 0, r
