"""Grad-weight with both operands shared by four filter tiles, on layers that take this path, against the fp64 oracle: row
groups and position chunks that are full, ragged and wrap, 2, 3 and 4 position tiles per workgroup, slices whose last round
is partial, planes of any remainder.  Bar: the suite's 2e-5 of the largest value (dw is binary32 in both data types); and the
error's 2-norm, which grows with the square root of the number of columns, 2**-24 * sqrt(N*H*W / 16) for one rounding per K group
of 16 columns, with a factor of 4 for the six products of a group."""
import numpy as np
import pytest
import torch

import paper_2101_00745_amd as S
import scc_workloads as Wk
from oracle import scc_oracle as O

CASES = [("f32", (330, 120, 500, 11, 9, 2, 0.33)),      # 99 pixels: the last group of a sample overlaps; 5 row groups, the last of 88 rows
         ("f32", (100, 104, 400, 23, 22, 1, 0.3)),      # walks once around the circle, entered past its end; last chunk of 8 positions
         ("f32", (37, 336, 330, 20, 41, 1, 0.5)),       # last row group of 74 rows; three chunks
         ("f32", (131, 96, 380, 30, 30, 2, 0.5)),       # 24 channels between starts; one chunk of 72 positions or more
         ("bf16", (330, 120, 500, 11, 9, 2, 0.33)), ("bf16", (100, 104, 400, 23, 22, 1, 0.3)),
         ("bf16", (37, 336, 330, 20, 41, 1, 0.5)), ("bf16", (131, 96, 380, 30, 30, 2, 0.5))]


def workspace(dtype, shape):
    return S.load().scc_backward_weight_workspace_bytes(*shape, 0 if dtype == "f32" else 1)


@pytest.mark.parametrize("dtype,shape", CASES)
def test_layers_here_take_the_path(dtype, shape):
    # the per-tile kernel cuts the columns into at most 256 slices of all tiles and asks for 4 MiB at most
    assert 4 << 20 < workspace(dtype, shape) <= S.scc.STATIC_SCRATCH_BYTES


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,shape", CASES)
def test_parity_and_repeat(dtype, shape):
    N, Cin, Cout, H, W, cg, co = shape
    layer = Wk.Layer("shared_weight", 9, N=N, Cin=Cin, Cout=Cout, H=H, W=W, cg=cg, co=co)
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    xd, wd, dyd = (torch.from_numpy(a).to(td).cuda() for a in Wk.make_inputs(layer))
    ref = O.backward_weight(xd.float().cpu().numpy(), dyd.float().cpu().numpy(), cg, co)
    dw = S.scc_backward_weight(xd, dyd, cg, co)
    got = dw.cpu().numpy().astype(np.float64)
    assert np.max(np.abs(got - ref)) <= 2e-5 * np.max(np.abs(ref))
    assert np.linalg.norm(got - ref) <= 4 * 2.0 ** -24 * np.sqrt(N * H * W / 16) * np.linalg.norm(ref)
    assert torch.equal(dw, S.scc_backward_weight(xd, dyd, cg, co))
    static = torch.empty_like(dw)
    S.scc_backward_weight_static(xd, dyd, cg, co, static)       # the same kernels on the library's own buffer
    assert torch.equal(dw, static)


# (dtype, layer) of scc_backward with both gradients in one launch; the first two as above, then: 64-column tiles beside
# slices of a few rounds; grad-input blocks of 16 channels in the last row group
BOTH = [("f32", (330, 120, 500, 11, 9, 2, 0.33)), ("bf16", (100, 104, 400, 23, 22, 1, 0.3)),
        ("f32", (64, 512, 1000, 7, 7, 2, 0.33)), ("bf16", (64, 512, 1000, 7, 7, 2, 0.33)),
        ("f32", (40, 272, 270, 28, 29, 1, 0.5)), ("bf16", (37, 336, 330, 20, 41, 1, 0.5)), ("f32", (95, 376, 376, 9, 9, 1, 0.33))]
BELOW = ("f32", (64, 512, 1000, 7, 7, 2, 0.33))      # fp32 needs more fetches than this layer's for the launch to pay


def backward_workspace(dtype, shape):
    return S.load().scc_backward_workspace_bytes(*shape, 0 if dtype == "f32" else 1)


@pytest.mark.parametrize("dtype,shape", [c for c in BOTH if c != BELOW])
def test_layers_here_take_one_launch(dtype, shape):
    # its workspace holds the packed weights as well: 16-position groups x 128 rows x 16 positions x (3 pieces or 1) of 2 bytes
    Cin, Cout = shape[1], shape[2]
    assert backward_workspace(dtype, shape) >= 8 * 4 * Cout * (Cin // shape[5]) + Cin * Cin // shape[5] * (6 if dtype == "f32" else 2)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,shape", BOTH)
def test_both_gradients_in_one_launch(dtype, shape):
    N, Cin, Cout, H, W, cg, co = shape
    layer = Wk.Layer("both", 9, N=N, Cin=Cin, Cout=Cout, H=H, W=W, cg=cg, co=co)
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    xd, wd, dyd = (torch.from_numpy(a).to(td).cuda() for a in Wk.make_inputs(layer))
    x, w, dy = (t.float().cpu().numpy() for t in (xd, wd, dyd))
    dx, dw = S.scc_backward(xd, dyd, wd, cg, co)
    ref_dx, ref_dw = O.backward_input(dy, w, Cin, cg, co), O.backward_weight(x, dy, cg, co)
    assert np.max(np.abs(dx.float().cpu().numpy() - ref_dx)) <= (2e-5 if dtype == "f32" else 1e-2) * np.max(np.abs(ref_dx))
    assert np.max(np.abs(dw.cpu().numpy() - ref_dw)) <= 2e-5 * np.max(np.abs(ref_dw))
    dx2, dw2 = S.scc_backward(xd, dyd, wd, cg, co)
    assert torch.equal(dx, dx2) and torch.equal(dw, dw2)
    # the same operands one float off their 16-byte alignment: same kernels, same bits
    shifted = [torch.empty(t.numel() + 1, dtype=t.dtype, device="cuda")[1:].view(t.shape).copy_(t) for t in (xd, dyd, wd)]
    dx3, dw3 = S.scc_backward(*shifted, cg, co)
    assert torch.equal(dx, dx3) and torch.equal(dw, dw3)


@pytest.mark.gpu
@pytest.mark.parametrize("which", ["backward_weight", "backward"])
@pytest.mark.parametrize("shape", [s for d, s in CASES if d == "f32"])
def test_products_are_binary32_to_the_end_of_the_exponent_range(shape, which):
    """dy of magnitude 2**-124 to 2**-123: normal numbers whose low halves no bf16 holds.  A product of cut pieces is off by up to
    2**-10 there; binary32 products keep the bar of test_parity_and_repeat."""
    N, Cin, Cout, H, W, cg, co = shape
    gen = torch.Generator(device="cuda").manual_seed(4)
    x = torch.randn(N, Cin, H, W, generator=gen, device="cuda") * 2.0 ** 60
    dy = torch.rand(N, Cout, H, W, generator=gen, device="cuda") + 1
    dy = dy * (torch.randint(0, 2, dy.shape, generator=gen, device="cuda") * 2 - 1) * 2.0 ** -62 * 2.0 ** -62
    ref = O.backward_weight(x.cpu().numpy(), dy.cpu().numpy(), cg, co)
    if which == "backward":
        dw = S.scc_backward(x, dy, torch.randn(Cout, Cin // cg, generator=gen, device="cuda"), cg, co)[1]
    else:
        dw = S.scc_backward_weight(x, dy, cg, co)
    got = dw.cpu().numpy().astype(np.float64)
    assert np.linalg.norm(got - ref) <= 4 * 2.0 ** -24 * np.sqrt(N * H * W / 16) * np.linalg.norm(ref)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,shape", CASES)
def test_an_infinite_gradient_stays_infinite(dtype, shape):
    N, Cin, Cout, H, W, cg, co = shape
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    gen = torch.Generator(device="cuda").manual_seed(4)
    x = (torch.rand(N, Cin, H, W, generator=gen, device="cuda") + 1).to(td)
    dy = torch.randn(N, Cout, H, W, generator=gen, device="cuda").to(td)
    dy[N // 2, Cout // 3, H - 1, W - 1] = float("inf")
    dw = S.scc_backward_weight(x, dy, cg, co)
    assert bool((dw[Cout // 3] == float("inf")).all())


# a wavefront's share of the columns, in the per-tile kernel and in a slice of the launch of both: bf16 layers whose 256 or 512
# workgroups alone would cut them into fewer slices
@pytest.mark.gpu
@pytest.mark.parametrize("dtype,shape", [("bf16", (30, 640, 640, 32, 32, 4, 0.0)), ("bf16", (68, 288, 288, 32, 32, 2, 0.0)),
                                         ("bf16", (64, 512, 1024, 7, 7, 2, 0.33)), ("f32", (64, 2048, 500, 16, 16, 1, 0.5))])
def test_sums_are_no_longer_than_the_per_tile_kernels(dtype, shape):
    """The error of dw against binary64 with the queried workspace and with the least one, which the per-tile kernel runs on.  Both
    are sums of some 10**5 roundings: 8 % between them is three times what their estimates scatter."""
    N, Cin, Cout, H, W, cg, co = shape
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    gen = torch.Generator(device="cuda").manual_seed(6)
    x, dy = (torch.randn(N, c, H, W, generator=gen, device="cuda").to(td) for c in (Cin, Cout))
    w = torch.randn(Cout, Cin // cg, generator=gen, device="cuda").to(td)
    L, step, _ = S.scc_window_params(Cin, Cout, cg, co)
    every = dy.double().transpose(0, 1).reshape(Cout, -1) @ x.double().transpose(0, 1).reshape(Cin, -1).t().contiguous()
    index = (torch.arange(Cout, device="cuda")[:, None] * step + torch.arange(L, device="cuda")) % Cin
    ref = every.gather(1, index)

    def error(bytes_):
        ws = torch.empty(bytes_, dtype=torch.uint8, device="cuda")
        return float((S.scc_backward(x, dy, w, cg, co, workspace=ws)[1].double() - ref).norm())

    need = backward_workspace(dtype, shape)
    assert need > 6 << 20
    assert error(need) <= 1.08 * error(6 << 20)      # 6 MiB: the most the per-tile kernel asks for, less than the launch of both


@pytest.mark.parametrize("dtype,shape", [("f32", (16, 768, 1533, 7, 7, 1, 0.5)), ("bf16", (4, 2048, 2048, 7, 7, 1, 0.5)),
                                         ("f32", (4, 2048, 2048, 7, 7, 1, 0.5))])
def test_few_columns_and_many_weights_are_not_cut_into_copies_of_dw(dtype, shape):
    assert backward_workspace(dtype, shape) == 0
