"""A block's training call in native code: the results of nn.DWSCCFunction, and DWSCCFunction itself for whatever is not plain."""
import pytest
import torch

from paper_2101_00745_amd import nn as N
from paper_2101_00745_amd import scc as B


def tensors(dtype=torch.float32, Cin=32, Cout=48, H=8, stride=1, grads=(True, True, True)):
    gen = torch.Generator(device="cuda").manual_seed(6)
    t = [torch.randn(*d, generator=gen, device="cuda").to(dtype).requires_grad_(g)
         for d, g in zip(((5, Cin, H, H), (Cin, 3, 3), (Cout, Cin // 2)), grads)]
    return t + [torch.randn(5, Cout, (H - 1) // stride + 1, (H - 1) // stride + 1, generator=gen, device="cuda").to(dtype)]


def native(*args):
    return B._load_native().dw_block(*args)


def grads(f, x, k, w, dy, stride):
    y = f(x, k, w, 2, 0.5, stride)
    return [y.detach()] + list(torch.autograd.grad(y, (x, k, w), dy))


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("Cin,Cout,H,stride", [(32, 48, 8, 1), (256, 512, 4, 1), (64, 61, 9, 2), (64, 128, 2, 1)])
def test_results_are_the_python_functions(dtype, Cin, Cout, H, stride):
    x, k, w, dy = tensors(dtype, Cin, Cout, H, stride)
    assert native(x, k, w, 2, 0.5, stride) is not None
    want = grads(N.DWSCCFunction.apply, x, k, w, dy, stride)
    for other in (dy, dy.clone(memory_format=torch.channels_last)):     # a gradient of other strides is made dense
        for a, b in zip(grads(N.dw_scc, x, k, w, other, stride), want):
            assert torch.equal(a, b) and a.dtype == b.dtype and a.is_contiguous()
    y = N.dw_scc(x, k, w, 2, 0.5, stride)
    assert not y._is_view()
    y.relu_().sum().backward()                                          # in place behind it, and a gradient of stride 0
    z = torch.relu(N.DWSCCFunction.apply(*(t.detach().requires_grad_() for t in (x, k, w)), 2, 0.5, stride))
    assert torch.equal(y.detach(), z.detach())


@pytest.mark.gpu
def test_what_is_not_plain_takes_the_python_function():
    x, k, w, dy = tensors()
    assert native(x, k, w, 2, 0.5, 1) is not None
    with torch.no_grad():
        assert native(x, k, w, 2, 0.5, 1) is None and not N.dw_scc(x, k, w, 2, 0.5).requires_grad
    for part in ((False, True, True), (True, False, True), (True, True, False), (False, False, False)):
        t = tensors(grads=part)[:3]
        assert native(*t, 2, 0.5, 1) is None
        y = N.dw_scc(*t, 2, 0.5)
        assert y.requires_grad == any(part)
        if any(part):
            y.backward(dy)
            assert [a.grad is not None for a in t] == list(part)
    assert native(x.transpose(2, 3), k, w, 2, 0.5, 1) is None and native(x, k, w, 2, 0, 1) is None and native(x.cpu(), k, w, 2, 0.5, 1) is None
    with pytest.raises(B.SccError):
        N.dw_scc(x, k, w, 2, 1.5)
    with pytest.raises(RuntimeError):                                   # no rule for functional transforms, as before
        torch.func.grad(lambda t: N.dw_scc(t, k, w, 2, 0.5).sum())(x)
    with pytest.raises(RuntimeError):
        torch.func.vmap(lambda t: N.dw_scc(t, k, w, 2, 0.5))(x[None])
    with torch.autograd.forward_ad.dual_level(), pytest.raises(RuntimeError):
        N.dw_scc(torch.autograd.forward_ad.make_dual(x, torch.ones_like(x)), k, w, 2, 0.5)


@pytest.mark.gpu
def test_hooks_checkpoints_and_misuse():
    x, k, w, dy = tensors()
    want = grads(N.DWSCCFunction.apply, x, k, w, dy, 1)[1:]
    seen = []
    with torch.autograd.graph.saved_tensors_hooks(lambda t: (seen.append(t.shape), t.cpu())[1], lambda t: t.cuda()):
        y = N.dw_scc(x, k, w, 2, 0.5)
    assert seen == [x.shape, k.shape, w.shape]
    got = [torch.autograd.grad(y, (x, k, w), dy, retain_graph=True), torch.autograd.grad(y, (x, k, w), dy)]
    with torch.autograd.graph.saved_tensors_hooks(lambda t: t, lambda t: t.transpose(0, 1).contiguous().transpose(0, 1)):
        y = N.dw_scc(x, k, w, 2, 0.5)
    with pytest.raises(ValueError, match="contiguous"):                 # what the general way says of such tensors
        torch.autograd.grad(y, x, dy)
    y = torch.utils.checkpoint.checkpoint(N.dw_scc, x, k, w, 2, 0.5, use_reentrant=False)
    got.append(torch.autograd.grad(y, (x, k, w), dy))
    for g in got:
        assert all(torch.equal(a, b) for a, b in zip(g, want))
    y = N.dw_scc(x, k, w, 2, 0.5)
    y.backward(dy)
    with pytest.raises(RuntimeError, match="second time"):
        y.backward(dy)
    y = N.dw_scc(x, k, w, 2, 0.5)
    with torch.no_grad():
        w += 1
    with pytest.raises(RuntimeError, match="modified by an inplace"):
        y.backward(dy)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        a = grads(N.dw_scc, x, k, w, dy, 1)
        b = grads(N.DWSCCFunction.apply, x, k, w, dy, 1)
    torch.cuda.current_stream().wait_stream(side)
    assert all(torch.equal(p, q) for p, q in zip(a, b))
