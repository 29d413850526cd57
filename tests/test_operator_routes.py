"""What the operator does under tracing, function transforms and saved-tensor hooks, where the library's calls are not
seen by PyTorch.  Runs without a GPU: the forward call is a stand-in that copies V's memory to O, the backward call one
that copies dO's to dV."""
import ctypes
import warnings

import pytest
import torch

import paper_2602_13515_amd as spa2
from paper_2602_13515_amd import autograd, binding

B, H, N, D = 1, 2, 130, 64
NBYTES = B * H * N * D * 2


class _Library:
    """The real library with the launching calls replaced."""

    def __init__(self, lib):
        self._lib = lib

    def __getattr__(self, name):
        return getattr(self._lib, name)

    @staticmethod
    def spa2_fwd(q, k, v, shape, pattern, scale, o, o_res, lse, ws, ws_bytes, stream):
        ctypes.memmove(o, v, NBYTES)
        return 0

    @staticmethod
    def spa2_bwd(q, k, v, o, o_res, d_o, lse, shape, pattern, scale, dq, dk, dv, ws, ws_bytes, stream):
        for out in (dq, dk):
            ctypes.memset(out, 0, NBYTES)
        ctypes.memmove(dv, d_o, NBYTES)
        return 0


@pytest.fixture(autouse=True)
def _stand_in(monkeypatch):
    lib = _Library(binding._load())
    monkeypatch.setattr(binding, "_load", lambda: lib)
    monkeypatch.setattr(binding, "_stream", lambda x: 0)
    monkeypatch.setattr(autograd, "_check_inputs", lambda q, k, v: None)      # (it asks for CUDA tensors)


def _qkv(seed):
    g = torch.Generator().manual_seed(seed)
    return [torch.randn((B, H, N, D), generator=g).bfloat16() for _ in range(3)]


def _attention(q, k, v):
    return spa2.sparge_attn2(q, k, v, 0.5, 0.5, pattern=binding.alloc_pattern(B, H, N, q.device))


@pytest.mark.parametrize("traced_with_grad", [False, True])
@pytest.mark.parametrize("replay_needs_grad", [False, True])
def test_traced_call_runs_on_the_inputs_of_the_replay(traced_with_grad, replay_needs_grad):
    with warnings.catch_warnings(), torch.set_grad_enabled(traced_with_grad):
        warnings.simplefilter("ignore")
        traced = torch.jit.trace(_attention, _qkv(1), check_trace=False)
    for seed in (2, 3):
        q, k, v = _qkv(seed)
        v.requires_grad_(replay_needs_grad)
        o = traced(q, k, v)
        assert torch.equal(o.detach(), v.detach())
        if replay_needs_grad:
            do = torch.full_like(v, 0.5)
            (dv,) = torch.autograd.grad(o, v, do)
            assert torch.equal(dv, do)


@pytest.mark.parametrize("transform", ["vmap", "grad", "functionalize"])
def test_function_transforms_are_refused(transform):
    """Also where the transformed tensors are not the operator's inputs."""
    q, k, v = _qkv(4)
    calls = {
        "vmap": lambda: torch.func.vmap(lambda x: _attention(q, k, v) + x)(torch.ones(3)),
        "grad": lambda: torch.func.grad(lambda x: (_attention(q, k, v).float() * x).sum())(torch.tensor(1.0)),
        "functionalize": lambda: torch.func.functionalize(lambda x: _attention(q, k, v) + x)(torch.ones(3, 1, 1, 1)),
    }
    with pytest.raises(RuntimeError):
        calls[transform]()


@pytest.mark.parametrize("grad", [False, True])
def test_inputs_with_tangents_are_refused(grad):
    import torch.autograd.forward_ad as fwad
    q, k, v = _qkv(5)
    with torch.set_grad_enabled(grad), fwad.dual_level():
        assert torch.equal(_attention(q, k, v), v)
        with pytest.raises(RuntimeError):
            _attention(q, k, fwad.make_dual(v, torch.ones_like(v)))


def _relaid(x):
    """The same values in memory of another layout (what a hook that packs with .contiguous() makes of a view)."""
    return x.transpose(1, 2).contiguous().transpose(1, 2)


@pytest.mark.parametrize("which", ["q", "k", "v", "o", "o_res", "lse"])
def test_saved_tensors_that_come_back_in_another_layout_are_refused(which):
    """The backward kernels take one stride triple for all token tensors: a saved-tensor hook that changes one of them
    must not be read through the strides of another."""
    n = 0

    def pack(x):
        nonlocal n
        n += 1                                        # saved in this order: q, k, v, o, o_res, lse
        return _relaid(x.detach()) if n - 1 == ("q", "k", "v", "o", "o_res", "lse").index(which) else x.detach()

    q, k, v = (t.requires_grad_(True) for t in _qkv(6))
    with torch.autograd.graph.saved_tensors_hooks(pack, lambda x: x):
        o = _attention(q, k, v)
    assert n == 6
    with pytest.raises(ValueError):
        o.backward(torch.ones_like(o))


def test_saved_tensors_that_come_back_as_copies_are_accepted():
    q, k, v = (t.requires_grad_(True) for t in _qkv(7))
    with torch.autograd.graph.saved_tensors_hooks(lambda x: x.detach().clone(), lambda x: x.clone()):
        o = _attention(q, k, v)
    (dv,) = torch.autograd.grad(o, v, torch.ones_like(o))
    assert torch.equal(dv, torch.ones_like(v))


@pytest.mark.parametrize("change", ["double", "shorter"])
def test_log_sum_exp_that_comes_back_as_something_else_is_refused(change):
    """It is read as B * H * N fp32 numbers, whatever a saved-tensor hook made of it."""
    as_else = {"double": lambda x: x.double(), "shorter": lambda x: x[..., :-1].contiguous()}[change]
    q, k, v = (t.requires_grad_(True) for t in _qkv(8))
    with torch.autograd.graph.saved_tensors_hooks(lambda x: x.detach(), lambda x: as_else(x) if x.dim() == 3 else x):
        o = _attention(q, k, v)
    with pytest.raises(ValueError):
        o.backward(torch.ones_like(o))


def test_log_sum_exp_that_comes_back_flat_is_accepted():
    q, k, v = (t.requires_grad_(True) for t in _qkv(9))
    with torch.autograd.graph.saved_tensors_hooks(lambda x: x.detach(), lambda x: x.flatten() if x.dim() == 3 else x):
        o = _attention(q, k, v)
    (dv,) = torch.autograd.grad(o, v, torch.ones_like(o))
    assert torch.equal(dv, torch.ones_like(v))
