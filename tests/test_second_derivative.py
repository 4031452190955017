"""Gradients taken with create_graph: they are what they are without it, and whoever differentiates them is told that there is no
second derivative, through the native block as through the Python functions.  (As plain results they would be constants, and a
penalty on them would be lost without a word.)"""
import pytest
import torch

from paper_2101_00745_amd import nn as N

CG, CO = 2, 0.5
KINDS = ["scc", "dw_scc", "DWSCCFunction"]


def call(kind, x, k, w):
    if kind == "scc":
        return N.scc(x, w, CG, CO)
    return N.dw_scc(x, k, w, CG, CO) if kind == "dw_scc" else N.DWSCCFunction.apply(x, k, w, CG, CO, 1)


def check(kind, device):
    gen = torch.Generator().manual_seed(5)
    x, k, w, dy = (torch.randn(*d, generator=gen).to(device) for d in ((3, 8, 4, 4), (8, 3, 3), (12, 4), (3, 12, 4, 4)))
    wanted = [t.requires_grad_() for t in ((x, w) if kind == "scc" else (x, k, w))]
    plain = torch.autograd.grad(call(kind, x, k, w), wanted, dy)
    assert not any(g.requires_grad for g in plain)
    # whatever of them asks for it, gradients that do not depend on dy's graph among them
    for grad_of_dy in (False, True):
        dy = dy.detach().requires_grad_(grad_of_dy)
        got = torch.autograd.grad(call(kind, x, k, w), wanted, dy, create_graph=True)
        for g, want in zip(got, plain):
            assert torch.equal(g, want) and g.requires_grad and not g._is_view()
            with pytest.raises(RuntimeError, match="second derivative"):
                (g.square().sum() + w.square().sum()).backward(retain_graph=True)
            assert torch.equal(g.mul_(2).detach(), want * 2)
    for t in wanted:
        t.grad = None
    call(kind, x, k, w).backward(dy, create_graph=True)                   # never differentiated again: served as ever
    assert all(torch.equal(t.grad, g) for t, g in zip(wanted, plain))
    for skip in range(len(wanted)):                                       # a tensor that wants none
        wanted[skip].requires_grad_(False)
        rest = [t for t in wanted if t.requires_grad]
        got = torch.autograd.grad(call(kind, x, k, w), rest, dy, create_graph=True)
        for g in got:
            with pytest.raises(RuntimeError, match="second derivative"):
                g.sum().backward(retain_graph=True)
        wanted[skip].requires_grad_(True)


@pytest.mark.parametrize("kind", KINDS)
def test_without_a_gpu(kind, monkeypatch):
    """The Python functions over stand-ins of the library's calls: windows as a dense matrix, the stage as a grouped convolution."""
    conv = torch.nn.functional.conv2d

    def dense(w, Cin):
        L, step, _ = N._scc.scc_window_params(Cin, w.shape[0], CG, CO)
        at = (torch.arange(w.shape[0])[:, None] * step + torch.arange(L)) % Cin
        return torch.zeros(w.shape[0], Cin).scatter(1, at, w)

    def block(x, k, w):
        z = conv(x, k[:, None], padding=1, groups=k.shape[0]) if k is not None else x
        return conv(z, dense(w, z.shape[1])[:, :, None, None])

    def grads(x, k, w, dy):
        with torch.enable_grad():
            t = [a.detach().requires_grad_() for a in (x, k, w) if a is not None]
            return torch.autograd.grad(block(t[0], t[1] if k is not None else None, t[-1]), t, dy.detach())

    class NoNative:
        dw_block = staticmethod(lambda *args: None)
    stand_ins = dict(_native=NoNative, scc_forward=lambda x, w, cg, co: block(x, None, w).detach(),
                     scc_dw_forward=lambda x, k, w, cg, co, s: block(x, k, w).detach(),
                     scc_backward=lambda x, dy, w, cg, co: grads(x, None, w, dy),
                     scc_backward_input=lambda dy, w, Cin, cg, co: grads(torch.zeros(dy.shape[0], Cin, *dy.shape[2:]), None, w, dy)[0],
                     scc_backward_weight=lambda x, dy, cg, co: grads(x, None, torch.zeros(dy.shape[1], x.shape[1] // cg), dy)[1],
                     _dw_backward=lambda x, k, w, dy, *rest: grads(x, k, w, dy),
                     scc_depthwise3x3_forward=lambda x, k, s: conv(x, k[:, None], padding=1, groups=k.shape[0]).detach(),
                     scc_depthwise3x3_backward=lambda x, k, dz, s, need_dx, need_dk: depthwise(x, k, dz))

    def depthwise(x, k, dz):
        with torch.enable_grad():
            t = [a.detach().requires_grad_() for a in (x, k)]
            return torch.autograd.grad(conv(t[0], t[1][:, None], padding=1, groups=k.shape[0]), t, dz.detach())
    for name, f in stand_ins.items():
        monkeypatch.setattr(N._scc, name, f)
    check(kind, "cpu")


@pytest.mark.gpu
@pytest.mark.parametrize("kind", KINDS)
def test_on_the_gpu(kind):
    check(kind, "cuda")
