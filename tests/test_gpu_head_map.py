"""Launches over many heads against one launch per head: every block of every head is taken exactly once, whichever way the
blocks of a head of that length are dealt to the XCDs."""

import numpy as np
import pytest
import torch

from paper_2602_13515_amd import workloads as wl

from gpu_util import dev, gpu_bwd, gpu_fwd, pattern_from_mask

pytestmark = pytest.mark.gpu


# row blocks (columns: twice that less one) on both sides of 32 and 128, where the way changes; lists of at most four
# entries, which no plan cuts, so that both sides add the same products in the same order
@pytest.mark.parametrize("H,Tm,d", [(5, 1, 128), (9, 11, 64), (5, 16, 128), (7, 17, 64), (9, 32, 128), (3, 33, 64),
                                    (3, 64, 64), (3, 65, 128), (2, 128, 64), (2, 129, 64)])
def test_heads_together_equal_heads_alone(H, Tm, d):
    N, Tn = 128 * Tm - 70, 2 * Tm - 1
    w = wl.Workload("heads", 1, H, N, d, 0.1, 0.5, "gaussian", True)
    q, k, v, do = (t.to(dev()) for t in wl.make_inputs(w, seed=3))
    rng = np.random.default_rng(11)
    mask = np.zeros((1, H, Tm, Tn), dtype=np.uint8)
    for _ in range(4):
        np.put_along_axis(mask, rng.integers(0, Tn, size=(1, H, Tm))[..., None], 1, axis=-1)
    mask *= (np.cumsum(mask, axis=2) <= 4).astype(np.uint8)
    pat = pattern_from_mask(mask, dev())
    o, lse, o_res = gpu_fwd(q, k, v, pat, residual=True)
    together = (o, lse) + tuple(gpu_bwd(q, k, v, o, do, lse, pat, o_res=o_res))
    for h in range(H):
        q1, k1, v1, do1 = (t[:, h:h + 1].clone(memory_format=torch.contiguous_format) for t in (q, k, v, do))
        pat1 = pattern_from_mask(np.ascontiguousarray(mask[:, h:h + 1]), dev())
        o1, lse1, res1 = gpu_fwd(q1, k1, v1, pat1, residual=True, split=False)
        alone = (o1, lse1) + tuple(gpu_bwd(q1, k1, v1, o1, do1, lse1, pat1, o_res=res1, split=False))
        for name, x, y in zip(("o", "lse", "dq", "dk", "dv"), together, alone):
            assert torch.equal(x[:, h:h + 1], y), (name, h)
