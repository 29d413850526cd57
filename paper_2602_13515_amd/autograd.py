"""`O = SpargeAttn2(Q, K, V, k%, p%)` (Sec. 4.3, Alg. 1) as a differentiable PyTorch operator.

A thin `torch.autograd.Function` over the three C calls: `spa2_mask` builds the block pattern from
Q and K, `spa2_fwd` runs the block-sparse attention, `spa2_bwd` returns dQ, dK, dV with the pattern
held constant (no gradient flows through the pooled scores, as in Alg. 2 where the mask is an
input of the attention call).  PyTorch allocates the buffers; every step runs in the HIP kernels.
"""
from __future__ import annotations

import functools
import importlib
import math
from typing import Optional, Tuple

import torch

from . import binding as _b


def _like(x: torch.Tensor) -> torch.Tensor:
    return torch.empty_strided(x.shape, x.stride(), dtype=x.dtype, device=x.device)


def _match(x: torch.Tensor, ref: torch.Tensor) -> torch.Tensor:
    """x with ref's strides (the kernels take one stride triple for all token tensors of a call)."""
    if x.stride() == ref.stride():
        return x
    y = _like(ref)
    y.copy_(x)
    return y


def _same_place(q: torch.Tensor, *others: torch.Tensor) -> None:
    """Shape, type and device of q (the strides are _match's)."""
    for t in others:
        if t.shape != q.shape or t.dtype != q.dtype or t.device != q.device:
            raise ValueError("all token tensors of one call share shape, strides, dtype and device")


def _check_inputs(q: torch.Tensor, k: torch.Tensor, v: torch.Tensor) -> None:
    for name, t in (("q", q), ("k", k), ("v", v)):
        if not t.is_cuda:
            raise ValueError(f"{name} must live on the GPU: the operator has no CPU path")
        if t.dtype != torch.bfloat16 or t.dim() != 4:
            raise ValueError(f"{name} must be a bf16 [B, H, N, d] view")
    if k.shape != q.shape or v.shape != q.shape:
        raise ValueError("self-attention: q, k, v share one shape")
    if q.stride(3) != 1:
        raise ValueError("the head dimension must be contiguous")


@functools.lru_cache(maxsize=None)
def _operator():
    """The operators in native code (csrc/operator.cpp)."""
    _b._load()
    try:
        return importlib.import_module(__package__ + "._operator")
    except ImportError as e:
        raise RuntimeError("_operator.so is missing or does not load: build it with `python -m paper_2602_13515_amd.build`") from e


def _plain(*tensors: torch.Tensor) -> bool:
    """Whether the native operators may take these tensors: plain CUDA tensors, outside tracing, compilation and function
    transforms (which have to see, or refuse, a Python autograd function)."""
    for t in tensors:
        if type(t) is not torch.Tensor and type(t) is not torch.nn.Parameter or not t.is_cuda:
            return False
    return (torch._C._get_tracing_state() is None and not torch._C._are_functorch_transforms_active()
            and not torch.compiler.is_compiling())


def build_pattern(q: torch.Tensor, k: torch.Tensor, k_frac: float, top_p: float,
                  scale: Optional[float] = None, columns: bool = True) -> _b.Pattern:
    """Hybrid Top-k + Top-p block pattern of (q, k) (Sec. 4.1; Alg. 1 steps 4-6).  The per-key-block lists are only
    read by the backward pass: `columns` False leaves them out."""
    B, H, N, d = q.shape
    scale = 1.0 / math.sqrt(d) if scale is None else float(scale)
    k = _match(k, q)
    lay = _b._layout_of(q)
    _same_place(q, k)
    pat = _b.alloc_pattern(B, H, N, q.device, columns=columns)
    ws = torch.empty(lay.mask_ws, dtype=torch.uint8, device=q.device)
    k_cnt = _b.spa2_topk_blocks(float(k_frac), lay.Tn)
    _b._mask_call(lay, q, k, k_cnt, float(top_p), scale, pat, ws, _b._stream(q))
    return pat


_side_streams = {}


def _side_stream(device: torch.device) -> torch.cuda.Stream:
    """One extra stream per device (default priority), made on first use, for `overlap_backward`."""
    key = torch.device(device).index
    if key not in _side_streams:
        _side_streams[key] = torch.cuda.Stream(device=device)
    return _side_streams[key]


def backward_two_streams(q, k, v, o, d_o, lse, pattern, scale, dq, dk, dv, workspace, o_res=None) -> None:
    """The backward pass as its three stage calls, with the dK/dV kernel on the current stream and the dQ kernel
    on a side stream at the same time.  Both read D, which the first call writes; they write different tensors,
    so the results are the bits `spa2_bwd` gives.  Each kernel fills what the other leaves idle at its end, which
    is little: on the 75,600-token layer the step takes 29.8 ms this way and 29.9 ms on one stream."""
    cur, side = torch.cuda.current_stream(q.device), _side_stream(q.device)
    _b.spa2_bwd_delta(o, d_o, workspace, o_res)
    fork = torch.cuda.Event()
    fork.record(cur)
    side.wait_event(fork)
    with torch.cuda.stream(side):
        _b.spa2_bwd_dq(q, k, v, d_o, lse, pattern, scale, dq, workspace)
    _b.spa2_bwd_dkdv(q, k, v, d_o, lse, pattern, scale, dk, dv, workspace)
    join = torch.cuda.Event()
    join.record(side)
    cur.wait_event(join)
    for t in (q, k, v, d_o, lse, dq, workspace):       # the caching allocator must not hand these out early
        t.record_stream(side)


def _forward(q, k, v, scale, pattern, residual: bool):
    """(k, v in q's layout), O, its bf16 residual (or None) and LSE."""
    k, v = _match(k, q), _match(v, q)
    lay = _b._layout_of(q)
    _same_place(q, k, v)
    o, o_res = _like(q), _like(q) if residual else None
    lse = torch.empty(q.shape[:3], dtype=torch.float32, device=q.device)
    ws_f = torch.empty(lay.fwd_ws, dtype=torch.uint8, device=q.device)   # long rows split
    _b._fwd_call(lay, q, k, v, pattern, scale, o, o_res, lse, ws_f, _b._stream(q))
    return k, v, o, o_res, lse


class _SpargeAttn2(torch.autograd.Function):
    """Calls without a backward pass to come go through here too: PyTorch does not see the library's calls, and this
    is what a trace replays and what refuses function transforms and inputs with tangents.  (Going round it would save
    them 4 us: 42 instead of 46 us on 1,000 tokens, two heads.)"""

    @staticmethod
    def forward(ctx, q, k, v, scale, pattern, overlap_backward=False, training=True):
        k, v, o, o_res, lse = _forward(q, k, v, scale, pattern, residual=training)
        if training:
            ctx.save_for_backward(q, k, v, o, o_res, lse)
            ctx.pattern, ctx.scale, ctx.overlap, ctx.device = pattern, scale, bool(overlap_backward), q.device
        return o

    @staticmethod
    def backward(ctx, d_o):
        q, k, v, o, o_res, lse = ctx.saved_tensors
        # (saved-tensor hooks may bring a tensor back in another layout, type or place)
        lay = _b._layout_of(q)
        if q.device != ctx.device:
            raise ValueError("saved token tensors come back on their GPU")
        if lse.device != q.device or lse.dtype != torch.float32 or lse.numel() != q.shape[:3].numel() or not lse.is_contiguous():
            raise ValueError("the log-sum-exp comes back as B * H * N contiguous fp32 numbers")
        d_o = _match(d_o.to(torch.bfloat16), q)
        _b._same_layout(q, k, v, o, o_res, d_o)
        dq, dk, dv = _like(q), _like(q), _like(q)
        ws = torch.empty(lay.bwd_ws, dtype=torch.uint8, device=q.device)
        if ctx.overlap:
            backward_two_streams(q, k, v, o, d_o, lse, ctx.pattern, ctx.scale, dq, dk, dv, ws, o_res)
        else:
            _b._bwd_call(lay, q, k, v, o, o_res, d_o, lse, ctx.pattern, ctx.scale, dq, dk, dv, ws, _b._stream(q))
        return dq, dk, dv, None, None, None, None


def sparge_attn2(q: torch.Tensor, k: torch.Tensor, v: torch.Tensor, k_frac: float, top_p: float,
                 scale: Optional[float] = None, pattern: Optional[_b.Pattern] = None,
                 return_pattern: bool = False, overlap_backward: bool = False):
    """Block-sparse attention on the blocks that the hybrid Top-k + Top-p rule selects.

    q, k, v: bf16 [B, H, N, d] views, d in {64, 128}, d contiguous; a [B, N, H, d] tensor is passed as
    `x.permute(0, 2, 1, 3)` without a copy.  k_frac, top_p in [0, 1].  `pattern`, when given, is used instead
    of building one from (q, k).  `overlap_backward` runs the two backward kernels at the same time on two
    streams (same results).  Returns O with q's shape and strides (and the pattern on request)."""
    if (pattern is not None or not return_pattern) and not overlap_backward and _plain(q, k, v):
        # The same in native code.  Passes (us): two heads, 1,000 tokens, sampling 46 -> 17; 2,048 tokens, forward and
        # backward 212 -> 82; 24 heads, 1,281 tokens 211 -> 116 (with the kernels' own changes).
        if scale is None:
            scale = 1.0 / math.sqrt(q.shape[-1]) if q.dim() and q.shape[-1] else 1.0      # (those are refused there)
        given = [] if pattern is None else [pattern.mask, pattern.row_cnt, pattern.row_idx, pattern.col_cnt,
                                            pattern.col_idx, pattern.row_order, pattern.col_order]
        o = _operator().attention(q, k, v, float(k_frac), float(top_p), float(scale), given)
        return (o, pattern) if return_pattern else o
    _check_inputs(q, k, v)
    scale = 1.0 / math.sqrt(q.shape[-1]) if scale is None else float(scale)
    # Without a backward pass to come (sampling) nobody reads the column lists or the output's residual: two kernels
    # and one tensor's writes fewer.  75,600 tokens, 40 heads: 4.85 -> 4.51 ms; 1,000 tokens, two heads: 69 -> 46 us.
    # (A trace may be replayed with gradients, whatever the mode it was recorded in.)
    training = (torch.is_grad_enabled() and (q.requires_grad or k.requires_grad or v.requires_grad)
                or torch.jit.is_tracing())
    if pattern is None:
        with torch.no_grad():
            pattern = build_pattern(q.detach(), k.detach(), k_frac, top_p, scale, columns=training or return_pattern)
    o = _SpargeAttn2.apply(q, k, v, scale, pattern, overlap_backward, training)
    return (o, pattern) if return_pattern else o


class SpargeAttn2(torch.nn.Module):
    """Attention core with fixed k% and p% (the appendix on hyper-parameters uses Top-k = 0.03 with Top-p = 0.2 or
    0.16 for about 95 % sparsity)."""

    def __init__(self, k_frac: float, top_p: float, scale: Optional[float] = None):
        super().__init__()
        self.k_frac, self.top_p, self.scale = float(k_frac), float(top_p), scale

    def forward(self, q: torch.Tensor, k: torch.Tensor, v: torch.Tensor) -> torch.Tensor:
        return sparge_attn2(q, k, v, self.k_frac, self.top_p, self.scale)

    def extra_repr(self) -> str:
        return f"k_frac={self.k_frac}, top_p={self.top_p}"
