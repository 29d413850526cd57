"""Column lists and launch order against the mask, for launches whose workgroups share 32 and 64 key blocks."""
import numpy as np
import pytest
import torch

import paper_2602_13515_amd as spa2

from gpu_util import Guarded, dev, guarded_pattern

pytestmark = pytest.mark.gpu


# launches of up to 128 workgroups of 64 key blocks are made with 32 each from 257 query blocks: one block; a block on either
# side of 32 and 64; T_m = 256 and 257; 126 and 135 workgroups; runs of more than 64 query blocks (T_m > 2048); 513 and 2049
# keys to rank
@pytest.mark.parametrize("B,H,Tm,Tn", [(1, 1, 1, 1), (1, 3, 16, 31), (2, 2, 17, 33), (1, 1, 33, 65), (1, 1, 2065, 4129), (2, 64, 8, 15),
                                       (1, 43, 65, 129), (1, 16, 256, 512), (1, 3, 257, 513), (1, 14, 257, 514),
                                       (1, 15, 257, 514), (1, 1, 1025, 2049)])
def test_columns_and_order_of_a_mask(B, H, Tm, Tn):
    N = min(128 * Tm, 64 * Tn)
    assert (-(-N // 128), -(-N // 64)) == (Tm, Tn)
    rng = np.random.default_rng(11)
    mask = rng.random((B, H, Tm, Tn)) < rng.random((B, H, 1, Tn)) ** 3      # columns of all lengths, some empty
    g = Guarded()
    pat = guarded_pattern(g, B, H, N, dev(), True)
    pat.mask.copy_(torch.from_numpy(mask.astype(np.uint8)))
    print(f"case B={B} H={H} Tm={Tm} Tn={Tn}", flush=True)
    spa2.spa2_mask_columns(torch.empty((B, H, N, 64), dtype=torch.bfloat16, device=dev()), pat)
    torch.cuda.synchronize()
    g.check("spa2_mask_columns")
    cnt, idx, order = (x.cpu().numpy().reshape(B * H, Tn, -1) for x in (pat.col_cnt, pat.col_idx, pat.col_order))
    chunk = -(-Tn // 8)
    places = [x * chunk + s for s in range(chunk) for x in range(8) if x * chunk + s < min((x + 1) * chunk, Tn)]
    for h, m in enumerate(mask.reshape(B * H, Tm, Tn)):
        length = m.sum(0)
        assert np.array_equal(cnt[h, :, 0], length)
        rows = np.nonzero(m.T)[1]
        taken = np.arange(Tm)[None, :] < length[:, None]
        assert np.array_equal(idx[h][taken], rows)
        want = np.empty(Tn, np.int64)
        want[places] = np.lexsort((np.arange(Tn), -length))
        assert np.array_equal(order[h, :, 0], want)
