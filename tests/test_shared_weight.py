"""Grad-weight with both operands shared by four filter tiles, on layers that take this path, against the fp64 oracle: row
groups and position chunks that are full, ragged and wrap, 2, 3 and 4 position tiles per workgroup, slices whose last round
is partial, planes of any remainder.  Bar: the suite's 2e-5 of the largest value (dw is binary32 in both data types); and the
error's 2-norm, 2**-24 * sqrt(N*H*W / 64): these layers are cut into at least 28 slices, a slice of n columns rounds its growing sum
n / 2 times (binary32, two columns a time) or n / 16 (bf16) by 2**-24 at most, which leaves 2**-24 * sqrt(n / 4) of the result
where partial sums grow as their square root, and sqrt(N*H*W / 112) of it for n = N*H*W / 28; the rest is for the sum over the slices."""
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


ANY, TILE, SHARED = 0, 1, 2                       # scc_weight_path of include/scc.h
TWO_PASSES, MERGED, BOTH_SHARED, FUSED = 0, 1, 2, 3   # scc_backward_paths


def path(which, dtype, shape, size):
    return getattr(S.load(), "scc_%s_path" % which)(*shape, 0 if dtype == "f32" else 1, size)


@pytest.mark.parametrize("dtype,shape", CASES)
def test_layers_here_take_the_path(dtype, shape):
    need = workspace(dtype, shape)
    assert need <= S.scc.STATIC_SCRATCH_BYTES
    # 6 MiB: the per-tile kernel's up to 510 tiles of 12 KiB
    assert [path("backward_weight", dtype, shape, size) for size in (need, need - 1, 6 << 20)] == [SHARED, TILE, TILE]


@pytest.mark.parametrize("shape,want", [((128, 256, 256, 16, 16, 4, 0.5, 0), (TILE, FUSED)), ((128, 256, 256, 16, 16, 4, 0.5, 1), (TILE, MERGED)),
                                        ((2, 8, 6, 3, 3, 2, 0.5, 0), (ANY, TWO_PASSES)), ((300, 32, 40, 1, 1, 2, 0.5, 0), (TILE, TWO_PASSES)),
                                        ((64, 1440, 510, 6, 6, 1, 0.5, 0), (TILE, MERGED)), ((64, 2048, 2048, 7, 7, 2, 0.5, 0), (SHARED, BOTH_SHARED)),
                                        ((190, 800, 69, 16, 16, 8, 0.0, 1), (SHARED, MERGED))])
def test_paths_of_other_layers(shape, want):
    lib = S.load()
    sizes = lib.scc_backward_weight_workspace_bytes(*shape), lib.scc_backward_workspace_bytes(*shape)
    assert (lib.scc_backward_weight_path(*shape, sizes[0]), lib.scc_backward_path(*shape, sizes[1])) == want


def test_paths_of_calls_that_are_refused():
    lib = S.load()
    for name in ("scc_backward_weight_path", "scc_backward_path"):
        call = getattr(lib, name)
        assert call(0, 8, 8, 4, 4, 2, 0.5, 0, 0) == -2 and call(1, 8, 8, 4, 4, 2, 1.5, 0, 0) == -3 and call(1, 8, 8, 4, 4, 2, 0.5, 7, 0) == -4
        assert call(128, 256, 256, 16, 16, 4, 0.5, 0, 1024) == -5


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
    assert np.linalg.norm(got - ref) <= 2.0 ** -24 * np.sqrt(N * H * W / 64) * np.linalg.norm(ref)
    assert torch.equal(dw, S.scc_backward_weight(xd, dyd, cg, co))
    static = torch.empty_like(dw)
    S.scc_backward_weight_static(xd, dyd, cg, co, static)       # the same kernels on the library's own buffer
    assert torch.equal(dw, static)


# (dtype, layer) of scc_backward with both gradients in one launch; the first two as above, then: 64-column tiles beside
# slices of a few rounds; grad-input blocks of 16 channels in the last row group
BOTH = [("f32", (330, 120, 500, 11, 9, 2, 0.33)), ("bf16", (100, 104, 400, 23, 22, 1, 0.3)),
        ("f32", (64, 512, 1000, 7, 7, 2, 0.33)), ("bf16", (64, 512, 1000, 7, 7, 2, 0.33)),
        ("f32", (40, 272, 270, 28, 29, 1, 0.5)), ("bf16", (37, 336, 330, 20, 41, 1, 0.5)), ("f32", (318, 200, 400, 5, 9, 1, 0.5)),
        ("bf16", (318, 200, 400, 5, 9, 1, 0.5))]
BELOW = (64, 512, 1000, 7, 7, 2, 0.33)               # saves too few fetches for the launch to pay


def backward_workspace(dtype, shape):
    return S.load().scc_backward_workspace_bytes(*shape, 0 if dtype == "f32" else 1)


@pytest.mark.parametrize("dtype,shape", BOTH)
def test_layers_here_take_one_launch(dtype, shape):
    need, least = backward_workspace(dtype, shape), 6 << 20
    assert path("backward", dtype, shape, need) == (MERGED if shape == BELOW else BOTH_SHARED)
    assert path("backward", dtype, shape, least) == MERGED


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
    assert np.linalg.norm(got - ref) <= 2.0 ** -24 * np.sqrt(N * H * W / 64) * np.linalg.norm(ref)


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
                                         ("bf16", (318, 200, 400, 5, 9, 1, 0.5)), ("f32", (64, 2048, 500, 16, 16, 1, 0.5))])
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


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,shape", [BOTH[0], BOTH[1], BOTH[6], BOTH[7]])
def test_both_gradients_in_a_graph(dtype, shape):
    """Every replay against the eager result, with other work and new inputs in between."""
    N, Cin, Cout, H, W, cg, co = shape
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    gen = torch.Generator(device="cuda").manual_seed(11)
    x, dy = (torch.randn(N, c, H, W, generator=gen, device="cuda").to(td) for c in (Cin, Cout))
    w = torch.randn(Cout, Cin // cg, generator=gen, device="cuda").to(td)
    dx, dw, alone = torch.empty_like(x), torch.empty(w.shape, device="cuda"), torch.empty(w.shape, device="cuda")
    ws = torch.empty(backward_workspace(dtype, shape), dtype=torch.uint8, device="cuda")

    def call():
        S.scc_backward(x, dy, w, cg, co, out_dx=dx, out_dw=dw, workspace=ws)
        S.scc_backward_weight_static(x, dy, cg, co, alone)

    call()                                               # code objects are loaded before the capture
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for _ in range(3):
        for t in (x, dy, w):
            t.copy_(torch.randn(t.shape, generator=gen, device="cuda"))
        for t in (dx, dw, alone):
            t.fill_(float("nan"))
        ws.fill_(255)
        graph.replay()
        torch.cuda.synchronize()
        want = S.scc_backward(x, dy, w, cg, co)
        assert torch.equal(dx, want[0]) and torch.equal(dw, want[1]) and torch.equal(alone, S.scc_backward_weight(x, dy, cg, co))
