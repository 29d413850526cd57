"""dK/dV launches whose workgroups draw their columns from a queue against the direct launch of the same columns."""

import numpy as np
import pytest
import torch

import paper_2602_13515_amd as spa2
from paper_2602_13515_amd import workloads as wl

from gpu_util import dev, gpu_bwd, gpu_fwd, pattern_from_mask

pytestmark = pytest.mark.gpu

# 2,048 columns go the direct way, 2,049 and more are drawn; ragged and full last blocks; columns of 0 to 4 entries, which
# no plan cuts, so that both ways add the same products in the same order
@pytest.mark.parametrize("B,H,N,d", [(2, 64, 1000, 128), (1, 683, 190, 64), (2, 40, 1700, 128), (1, 129, 1024, 64)])
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
    o, lse, o_res = gpu_fwd(q, k, v, pat, residual=True)
    queued = gpu_bwd(q, k, v, o, do, lse, pat, o_res=o_res)
    direct = gpu_bwd(q, k, v, o, do, lse, pat, o_res=o_res, split=False)
    again = gpu_bwd(q, k, v, o, do, lse, pat, o_res=o_res)
    for name, x, y, z in zip(("dq", "dk", "dv"), queued, direct, again):
        assert torch.equal(x, y), name
        assert torch.equal(x, z), name


# one, three and nine columns a head: no XCD is left without
@pytest.mark.parametrize("H,N,d", [(2100, 60, 64), (700, 190, 128), (240, 567, 64)])
def test_queue_over_heads_of_a_few_columns(H, N, d):
    g = torch.Generator().manual_seed(2)
    q, k, v, do = (torch.randn((1, H, N, d), generator=g).bfloat16().to(dev()) for _ in range(4))
    pat = spa2.alloc_pattern(1, H, N, dev())
    spa2.spa2_pattern_full(q, pat)
    o, lse, o_res = gpu_fwd(q, k, v, pat, residual=True)
    queued = gpu_bwd(q, k, v, o, do, lse, pat, o_res=o_res)
    direct = gpu_bwd(q, k, v, o, do, lse, pat, o_res=o_res, split=False)
    for name, x, y in zip(("dq", "dk", "dv"), queued, direct):       # (five entries a column at most: nothing is cut)
        assert torch.equal(x, y), name
