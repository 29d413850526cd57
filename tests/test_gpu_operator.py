"""The operators' native route (plain CUDA tensors) against the Python autograd functions behind the other calls."""
import ctypes

import pytest
import torch

import paper_2602_13515_amd as spa2
from paper_2602_13515_amd import autograd
from paper_2602_13515_amd import workloads as wl
from paper_2602_13515_amd.distill import _VelocityDistillationLoss, velocity_distillation_loss

from gpu_util import Guarded, dev, gpu_fwd, gpu_mask, guarded_pattern

pytestmark = pytest.mark.gpu

# 32 and 504 key blocks take no launch order, 513 and 632 do; a query block and a key block that end early; k and v in
# another layout than q
CASES = [(1, 2, 1000, 64, "bhnd"), (1, 1, 64 * 513, 64, "bhnd"), (4, 6, 1281, 128, "bnhd"), (2, 2, 10090, 128, "mixed")]


def _inputs(B, H, N, d, layout):
    w = wl.Workload("op", B, H, N, d, 0.1, 0.6, "lowrank", True)
    q, k, v, do = (t.to(dev()) for t in wl.make_inputs(w, seed=3))
    bnhd = lambda t: t.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)
    if layout == "bnhd":
        q, k, v, do = (bnhd(t) for t in (q, k, v, do))
    elif layout == "mixed":
        k = bnhd(k)
    return q, k, v, do


@pytest.mark.parametrize("B,H,N,d,layout", CASES)
def test_native_route_gives_the_bits_of_the_python_route(B, H, N, d, layout, monkeypatch):
    q, k, v, do = _inputs(B, H, N, d, layout)
    got, full = {}, spa2.build_pattern(q, k, 0.05, 0.3)
    for native in (True, False):
        if not native:
            monkeypatch.setattr(autograd, "_plain", lambda *t: False)
        with torch.no_grad():
            sampled = spa2.sparge_attn2(q, k, v, 0.1, 0.6)
        leaves = [t.detach().requires_grad_(True) for t in (q, k, v)]
        o = spa2.sparge_attn2(*leaves, 0.1, 0.6)
        assert ("CppNode" in o.grad_fn.name()) == native
        assert o.stride() == q.stride()
        got[native] = (sampled, o.detach(), *torch.autograd.grad(o, leaves, do))
        o = spa2.sparge_attn2(*leaves, 0.0, 0.0, pattern=full)
        got[native] += (o.detach(), *torch.autograd.grad(o, leaves, do))
    for a, b in zip(*got.values()):
        assert torch.equal(a, b)


# rows cut by the sizes alone (no plan) and by the plan: 16 and 17 heads of 32 blocks stand on either side of that rule; rows
# of one part, of two and of four, the last one short
@pytest.mark.parametrize("H,N,d", [(2, 513, 128), (1, 1000, 64), (2, 2048, 64), (16, 2048, 128), (17, 2048, 64), (3, 1281, 128)])
def test_small_layers_cut_rows_as_the_plan_does(H, N, d, monkeypatch):
    q, k, v, _ = _inputs(1, H, N, d, "bhnd")
    for k_frac in (0.3, 0.9, 1.0):
        with torch.no_grad():
            native = [spa2.sparge_attn2(q, k, v, k_frac, 0.0) for _ in range(2)]
            with monkeypatch.context() as m:
                m.setattr(autograd, "_plain", lambda *t: False)
                planned = spa2.sparge_attn2(q, k, v, k_frac, 0.0)
        assert torch.equal(native[0], planned) and torch.equal(native[1], planned), k_frac


@pytest.mark.parametrize("rows,dtype,reduction", [(1, torch.float32, "mean"), (777, torch.bfloat16, "batch")])
def test_native_loss_gives_the_bits_of_the_python_route(rows, dtype, reduction):
    g = torch.Generator().manual_seed(1)
    us, uf = (torch.randn((2, rows, 65), generator=g).to(dev(), dtype) for _ in range(2))
    a, b = us.clone().requires_grad_(True), us.clone().requires_grad_(True)
    loss = velocity_distillation_loss(a, uf, reduction)
    ref = _VelocityDistillationLoss.apply(b, uf, 1.0 / (us.numel() if reduction == "mean" else 2))
    assert torch.equal(loss, ref)
    (3.0 * loss).backward(); (3.0 * ref).backward()
    assert torch.equal(a.grad, b.grad)


# one element, less than a vector, vectors and a remainder, more than one round of the 2,048 workgroups
@pytest.mark.parametrize("n", [1, 3, 1029, 2048 * 256 * 4 + 5])
def test_loss_and_gradient_in_one_pass(n):
    g = torch.Generator().manual_seed(n)
    us, uf = (torch.randn(n, generator=g).to(dev()) for _ in range(2))
    weight = 0.7 / n
    new = lambda: torch.full((n,), float("nan"), device=dev())
    scalar = lambda x: torch.tensor(x, dtype=torch.float64, device=dev())
    ws = torch.empty(spa2.binding.spa2_vd_loss_workspace_bytes(), dtype=torch.uint8, device=dev())
    loss, ref_loss, grad, ref = scalar(0.0), scalar(0.0), new(), new()
    spa2.binding.spa2_vd_loss_and_grad(us, uf, weight, loss, grad, ws)
    spa2.binding.spa2_vd_loss(us, uf, weight, ref_loss, ws)
    assert abs(loss - ref_loss) <= 1e-12 * ref_loss          # fp64 sums in two orders
    for u in (1.0, 4.0, 0.3):
        got = grad.clone()
        spa2.binding.spa2_vd_rescale(got, weight, scalar(u))
        spa2.binding.spa2_vd_loss_grad(us, uf, weight, scalar(u), ref)
        if u != 0.3:      # 2 * 0.7 / n is within 2^-25 of its fp32 value for these n: powers of two give the same bits
            assert torch.equal(got, ref)
        else:      # on either side three roundings to fp32 of 2^-24 each: difference, factor or product, product
            assert ((got - ref).abs() <= 2.0 ** -22 * ref.abs()).all()


# factors 2 / n that are not fp32 numbers.  Two roundings of 2^-24 on either side: both products where the gradient is rescaled,
# factor and product where it is made for that upstream
@pytest.mark.parametrize("n", [1_000_003, 11, 22_369_627])
def test_rescaled_gradient_is_within_its_bound(n):
    g = torch.Generator(device=dev()).manual_seed(n)
    us, uf = (torch.randn(n, generator=g, device=dev()) for _ in range(2))
    weight = 1.0 / n
    grad, ref = torch.empty_like(us), torch.empty_like(us)
    loss = torch.zeros((), dtype=torch.float64, device=dev())
    ws = torch.empty(spa2.binding.spa2_vd_loss_workspace_bytes(), dtype=torch.uint8, device=dev())
    spa2.binding.spa2_vd_loss_and_grad(us, uf, weight, loss, grad, ws)
    exact = 2.0 * weight * (us - uf).double()
    for u in (1.0, 2.0, 4.0, 0.3, 65536.0):
        up = torch.tensor(u, dtype=torch.float64, device=dev())
        got = grad.clone()
        spa2.binding.spa2_vd_rescale(got, weight, up)
        spa2.binding.spa2_vd_loss_grad(us, uf, weight, up, ref)
        assert ((got - ref).abs() <= 2.0 ** -22 * ref.abs()).all(), u
        assert ((got.double() - u * exact).abs() <= 2.0 ** -23 * (u * exact).abs() * (1 + 1e-6)).all(), u
        if u == 1.0:
            assert torch.equal(got, grad) and torch.equal(got, ref)


def test_second_backward_pass_gets_a_gradient_of_its_own():
    us, uf = (torch.randn(4, 333, device=dev()) for _ in range(2))
    us.requires_grad_(True)
    loss = velocity_distillation_loss(us, uf)
    (first,) = torch.autograd.grad(loss, us, retain_graph=True)
    kept = first.clone()
    first.zero_()
    (second,) = torch.autograd.grad(loss, us)
    assert torch.equal(second, kept) and second.data_ptr() != first.data_ptr()


def test_native_route_refuses_what_the_python_route_refuses():
    q, k, v, do = _inputs(1, 2, 300, 64, "bhnd")
    call = lambda *t: spa2.sparge_attn2(*t, 0.1, 0.6)
    with pytest.raises(RuntimeError):
        torch.func.vmap(lambda x: call(q, k, v) + x)(torch.ones(3, device=dev()))
    for bad in ((q.cpu(), k, v), (q, k.cpu(), v), (q, k.float(), v), (q, k[:, :, :299], v), (q[0], k[0], v[0]),
                (q, k, v.transpose(2, 3).contiguous())):
        with pytest.raises(ValueError):
            call(*bad)
    rows = spa2.build_pattern(q, k, 0.1, 0.6, columns=False)       # no lists for the backward pass
    o = spa2.sparge_attn2(*(t.detach().requires_grad_(True) for t in (q, k, v)), 0.0, 0.0, pattern=rows)
    with pytest.raises(spa2.Spa2Error):
        o.backward(do)
    with pytest.raises(spa2.Spa2Error) as e:                       # head dimension 32
        call(*(t[..., :32].contiguous() for t in (q, k, v)))
    assert e.value.code < 0
    leaves = [t.detach().requires_grad_(True) for t in (q, k, v)]
    relaid = lambda x: x.transpose(1, 2).contiguous().transpose(1, 2) if x.dim() == 4 and x.data_ptr() == leaves[1].data_ptr() else x
    with torch.autograd.graph.saved_tensors_hooks(relaid, lambda x: x):      # k comes back in another layout
        o = call(*leaves)
    with pytest.raises(ValueError):
        o.backward(do)
    o = call(*leaves)
    o.backward(do)
    with pytest.raises(RuntimeError):                              # a second time without retain_graph
        o.backward(do)


# what the hooks make of the token tensors and of the log-sum-exp.  Nothing may be launched on these: the kernels would read
# host memory, rows through wrong strides, or past the end
BROUGHT_BACK = {
    "on the host": (lambda x: x.cpu(), lambda x: x.cpu()),
    "channels apart": (lambda x: x.transpose(2, 3).contiguous().transpose(2, 3), lambda x: x),
    "in fp32": (lambda x: x.float(), lambda x: x),
    "log-sum-exp on the host": (lambda x: x, lambda x: x.cpu()),
    "log-sum-exp in fp64": (lambda x: x, lambda x: x.double()),
    "log-sum-exp shorter": (lambda x: x, lambda x: x[..., :-1].contiguous()),
}


@pytest.mark.parametrize("change", BROUGHT_BACK)
@pytest.mark.parametrize("given", [False, True])
def test_native_backward_refuses_saved_tensors_of_another_place_or_kind(change, given):
    q, k, v, do = _inputs(1, 2, 300, 64, "bhnd")
    pattern = spa2.build_pattern(q, k, 0.1, 0.6) if given else None
    tokens, lse = BROUGHT_BACK[change]
    leaves = [t.detach().requires_grad_(True) for t in (q, k, v)]
    with torch.autograd.graph.saved_tensors_hooks(lambda x: x.detach(), lambda x: tokens(x) if x.dim() == 4 else lse(x)):
        o = spa2.sparge_attn2(*leaves, 0.1, 0.6, pattern=pattern)
    assert "CppNode" in o.grad_fn.name()
    # (an upstream gradient of other strides is copied to those of q, wherever q is)
    with pytest.raises(ValueError):
        o.backward(do.transpose(1, 2).contiguous().transpose(1, 2))


# 16 and 17 heads of 32 blocks stand on either side of the sizes that need no plan; ragged blocks; a row of one block
@pytest.mark.parametrize("H,N,d", [(16, 2048, 64), (17, 2048, 64), (2, 1000, 128), (1, 40, 128), (5, 10090, 64)])
@pytest.mark.parametrize("columns", [True, False])
def test_pattern_and_forward_in_a_workspace_of_exactly_the_reported_size(H, N, d, columns):
    """spa2_mask_fwd between guard zones against spa2_mask and spa2_fwd: same bits, nothing written outside a buffer."""
    q, k, v, _ = _inputs(1, H, N, d, "bhnd")
    tn = -(-N // 64)
    topk, scale = spa2.spa2_topk_blocks(0.3, tn), d ** -0.5
    lib, g = spa2.binding._load(), Guarded()
    lay = spa2.binding._layout_of(q)
    need = int(lib.spa2_mask_fwd_workspace_bytes(lay.ref))
    pat = guarded_pattern(g, 1, H, N, dev(), columns)
    new = lambda: g.alloc(q.shape, q.dtype, dev(), float("nan"))
    o, o_res, lse = new(), new(), g.alloc((1, H, N), torch.float32, dev(), float("nan"))
    ws = g.alloc((need,), torch.uint8, dev(), 0xA5)
    c = pat._c()
    call = lambda nbytes: lib.spa2_mask_fwd(q.data_ptr(), k.data_ptr(), v.data_ptr(), lay.ref, topk, 0.6, scale, ctypes.byref(c),
                                            o.data_ptr(), o_res.data_ptr(), lse.data_ptr(), ws.data_ptr(), nbytes,
                                            spa2.binding._stream(q))
    assert call(need - 1) == -6 and call(need) == 0
    torch.cuda.synchronize()
    g.check("spa2_mask_fwd")
    ref, _ = gpu_mask(q, k, topk, 0.6, scale, want_pbar=False, columns=columns)
    assert torch.equal(pat.mask, ref.mask) and torch.equal(pat.row_cnt, ref.row_cnt)
    for a, b in zip((o, lse, o_res), gpu_fwd(q, k, v, ref, scale, residual=True)):
        assert torch.equal(a, b)
    if columns:
        assert torch.equal(pat.col_cnt, ref.col_cnt) and torch.equal(pat.col_idx, ref.col_idx)


SAVED = ("q", "k", "v", "o", "o_res", "lse")         # in the order in which they are saved


@pytest.mark.parametrize("given", [False, True])
def test_native_backward_takes_saved_tensors_that_come_back_as_copies(given):
    q, k, v, do = _inputs(1, 3, 1281, 128, "bnhd")
    pattern = spa2.build_pattern(q, k, 0.1, 0.6) if given else None
    leaves = [t.detach().requires_grad_(True) for t in (q, k, v)]
    want = torch.autograd.grad(spa2.sparge_attn2(*leaves, 0.1, 0.6, pattern=pattern), leaves, do)
    packed = []
    pack = lambda x: (packed.append(x), x.detach().cpu())[1]
    unpack = lambda x: (x if x.dim() == 4 else x.flatten()).to(dev())          # (of the log-sum-exp only the numbers count)
    with torch.autograd.graph.saved_tensors_hooks(pack, unpack):
        o = spa2.sparge_attn2(*leaves, 0.1, 0.6, pattern=pattern)
    assert "CppNode" in o.grad_fn.name() and len(packed) == len(SAVED)
    del packed[:]
    for a, b in zip(torch.autograd.grad(o, leaves, do), want):
        assert torch.equal(a, b)


@pytest.mark.parametrize("which", SAVED)
def test_native_backward_refuses_each_saved_tensor_in_another_layout(which):
    q, k, v, do = _inputs(1, 2, 300, 64, "bhnd")
    leaves = [t.detach().requires_grad_(True) for t in (q, k, v)]
    count = []

    def pack(x):
        count.append(0)
        return (x.detach().transpose(1, 2).contiguous().transpose(1, 2) if SAVED[len(count) - 1] == which else x.detach())

    with torch.autograd.graph.saved_tensors_hooks(pack, lambda x: x):
        o = spa2.sparge_attn2(*leaves, 0.1, 0.6)
    assert "CppNode" in o.grad_fn.name() and len(count) == len(SAVED)
    with pytest.raises(ValueError):
        o.backward(do)


@pytest.mark.parametrize("early_stop", [True, False])
def test_native_route_under_non_reentrant_checkpoint(early_stop):
    """The recomputation is ended by an exception that the pack hook throws through the native call."""
    from torch.utils.checkpoint import checkpoint, set_checkpoint_early_stop
    q, k, v, do = _inputs(1, 2, 1000, 64, "bhnd")
    uf = torch.randn(q.shape, device=dev())
    leaves = [t.detach().requires_grad_(True) for t in (q, k, v)]
    layer = lambda a, b, c: spa2.sparge_attn2(2 * a, b, c, 0.1, 0.6)
    head = lambda x: velocity_distillation_loss(x.float(), uf)
    want = torch.autograd.grad(layer(*leaves), leaves, do)
    want_loss = torch.autograd.grad(head(layer(*leaves)), leaves)
    with set_checkpoint_early_stop(early_stop):
        o = checkpoint(layer, *leaves, use_reentrant=False)
        got = torch.autograd.grad(o, leaves, do)
        loss = checkpoint(lambda *t: head(layer(*t)), *leaves, use_reentrant=False)
        got_loss = torch.autograd.grad(loss, leaves)
    for a, b in zip((*got, *got_loss), (*want, *want_loss)):
        assert torch.equal(a, b)


def test_an_exception_of_a_pack_hook_leaves_the_native_call_as_it_is():
    class Refused(Exception):
        pass

    def refuse(x):
        raise Refused

    q, k, v, do = _inputs(1, 2, 300, 64, "bhnd")
    leaves = [t.detach().requires_grad_(True) for t in (q, k, v)]
    with pytest.raises(Refused), torch.autograd.graph.saved_tensors_hooks(refuse, lambda x: x):
        spa2.sparge_attn2(*leaves, 0.1, 0.6)
    spa2.sparge_attn2(*leaves, 0.1, 0.6).backward(do)
    assert all(bool(t.grad.isfinite().all()) for t in leaves)


def test_gradients_of_either_route_have_no_second_derivative(monkeypatch):
    q, k, v, do = _inputs(1, 2, 300, 64, "bhnd")
    for native in (True, False):
        if not native:
            monkeypatch.setattr(autograd, "_plain", lambda *t: False)
        leaves = [t.detach().requires_grad_(True) for t in (q, k, v)]
        grads = torch.autograd.grad(spa2.sparge_attn2(*leaves, 0.1, 0.6), leaves, do, create_graph=True)
        assert not any(g.requires_grad for g in grads), native
