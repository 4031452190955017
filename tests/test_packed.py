"""Forward and grad-input as a product with packed weights (scc_forward_ws, scc_backward_input_ws) against the fp64 oracle on
layers that take this path: row groups, column tiles, rounds and walks that are full, ragged or wrap; both tile widths;
planes of any remainder.  Bars: those of the suite (2e-5 of the largest value in fp32, 1e-2 in bf16)."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2101_00745_amd as S
import scc_workloads as Wk
from oracle import scc_oracle as O
from paper_2101_00745_amd import scc as B

BANDED = (130, 120, 500, 11, 9, 2, 0.33)     # 120 window starts x 5 filters, 100 of the 600 rows empty; 99 pixels
CIRCLE = (20, 104, 400, 46, 44, 1, 0.3)      # every window reaches every channel block: walks are once around the circle
NARROW = (64, 512, 1000, 7, 7, 2, 0.33)      # 64-column tiles; last row group of 104 rows; walk of 23 rounds
DENSE = (110, 336, 330, 16, 18, 1, 0.5)       # two windows x 165 filters; last row group of 74 rows
GAPS = (190, 320, 160, 37, 28, 4, 0.0)        # four windows side by side: grad-input's blocks see one or two of them
ROUND = (60, 96, 190, 30, 44, 4, 0.76)       # windows of 24 channels, 6 apart; a forward walk of two rounds
CASES = [("forward", "f32", s) for s in (BANDED, CIRCLE, NARROW, DENSE, ROUND)] + \
        [("forward", "bf16", s) for s in (BANDED, CIRCLE, NARROW, DENSE, ROUND)] + \
        [("backward_input", "f32", s) for s in (CIRCLE, DENSE, GAPS)] + \
        [("backward_input", "bf16", s) for s in (BANDED, CIRCLE, NARROW, DENSE, GAPS)]


def need(which, dtype, shape):
    return getattr(S.load(), "scc_%s_workspace_bytes" % which)(*shape, 0 if dtype == "f32" else 1)


@pytest.mark.parametrize("which,dtype,shape", CASES)
def test_layers_here_take_the_path_and_a_short_workspace_is_refused(which, dtype, shape):
    n = need(which, dtype, shape)
    assert n > 0
    call = getattr(S.load(), "scc_%s_ws" % which)
    fake, code = ctypes.c_void_p(0x1000), 0 if dtype == "f32" else 1
    for ws, size in ((0x1000, n - 1), (0x1010, n)):              # too small; not 256-byte aligned
        assert call(fake, fake, fake, *shape, code, ws, size, None) == -5
    assert call(fake, None, fake, *shape, code, 0x1000, n, None) == -1


@pytest.mark.gpu
@pytest.mark.parametrize("which,dtype,shape", CASES)
def test_parity(which, dtype, shape):
    N, Cin, Cout, H, W, cg, co = shape
    layer = Wk.Layer("packed", 9, N=N, Cin=Cin, Cout=Cout, H=H, W=W, cg=cg, co=co)
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    xd, wd, dyd = (torch.from_numpy(a).to(td).cuda() for a in Wk.make_inputs(layer))
    x, w, dy = (t.float().cpu().numpy() for t in (xd, wd, dyd))
    if which == "forward":
        got, ref = S.scc_forward(xd, wd, cg, co), O.forward(x, w, cg, co)
    else:
        got, ref = S.scc_backward_input(dyd, wd, Cin, cg, co), O.backward_input(dy, w, Cin, cg, co)
    err = np.max(np.abs(got.float().cpu().numpy() - ref)) / np.max(np.abs(ref))
    assert err <= (2e-5 if dtype == "f32" else 1e-2), err
    # without a workspace: the other kernels, the same definition
    out = torch.empty_like(got)
    src = xd if which == "forward" else dyd
    shp = shape + (0 if dtype == "f32" else 1,)
    assert getattr(S.load(), "scc_" + which)(src.data_ptr(), wd.data_ptr(), out.data_ptr(), *shp,
                                             torch.cuda.current_stream().cuda_stream) == 0
    err = np.max(np.abs(out.float().cpu().numpy() - ref)) / np.max(np.abs(ref))
    assert err <= (2e-5 if dtype == "f32" else 1e-2), err


def test_queries_of_bad_arguments_are_zero():
    for bad in ((0, 8, 8, 4, 4, 2, 0.5, 0), (1, 9, 8, 4, 4, 2, 0.5, 0), (1, 8, 8, 4, 4, 2, 1.5, 0), (1, 8, 8, 4, 4, 2, 0.5, 7)):
        assert B.load().scc_forward_workspace_bytes(*bad) == 0
        assert B.load().scc_backward_input_workspace_bytes(*bad) == 0


@pytest.mark.gpu
@pytest.mark.parametrize("which,dtype,shape", [CASES[0], CASES[7], CASES[10], CASES[15]])
def test_calls_with_out_allocate_nothing_and_a_workspace_can_be_handed_over(which, dtype, shape):
    N, Cin, Cout, H, W, cg, co = shape
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    gen = torch.Generator(device="cuda").manual_seed(8)
    src, dst = (Cin, Cout) if which == "forward" else (Cout, Cin)
    x = torch.randn(N, src, H, W, generator=gen, device="cuda").to(td)
    w = torch.randn(Cout, Cin // cg, generator=gen, device="cuda").to(td)
    out = torch.empty(N, dst, H, W, dtype=td, device="cuda")

    def call(**kw):
        return S.scc_forward(x, w, cg, co, **kw) if which == "forward" else S.scc_backward_input(x, w, Cin, cg, co, **kw)

    plain = call()
    before = torch.cuda.memory_stats()["allocation.all.allocated"]
    assert call(out=out) is out
    assert torch.cuda.memory_stats()["allocation.all.allocated"] == before
    bar = 2e-5 if dtype == "f32" else 1e-2
    assert float((out.float() - plain.float()).abs().max()) <= bar * float(plain.float().abs().max())
    query = S.scc_forward_workspace_bytes if which == "forward" else S.scc_backward_input_workspace_bytes
    ws = torch.empty(query(*shape, td), dtype=torch.uint8, device="cuda")
    before = torch.cuda.memory_stats()["allocation.all.allocated"]
    call(out=out, workspace=ws)
    assert torch.cuda.memory_stats()["allocation.all.allocated"] == before
    assert torch.equal(out, plain)
    with pytest.raises(S.SccError):
        call(out=out, workspace=ws[:-1])


# ---- the products of binary32 operands: six of the nine partial products of two three-way cuts ------------------------------
def cut(v):
    """The cut of split3 (scc_common.h): upper halves taken off one after the other."""
    top = lambda a: (a.view(np.uint32) & np.uint32(0xffff0000)).view(np.float32)
    hi = top(v)
    mid = top(v - hi)
    return [p.astype(np.float64) for p in (hi, mid, top((v - hi) - mid))]


def test_dropped_products_are_below_the_stated_bound():
    """include/scc.h: less than 2**-21 of the product, always toward zero; and not less than 2**-23."""
    rng = np.random.default_rng(3)
    a, b = (np.concatenate([rng.standard_normal(1 << 18), [1 + 2.0 ** -7 - 2.0 ** -23]]).astype(np.float32) for _ in range(2))
    (ah, am, al), (bh, bm, bl) = cut(a), cut(b)
    exact = a.astype(np.float64) * b
    assert np.array_equal((ah + am) + al, a) and np.array_equal((bh + bm) + bl, b)
    loss = (exact - (ah * bh + (ah * bm + am * bh) + (am * bm + ah * bl + al * bh))) / exact
    assert loss.min() >= 0 and 2.0 ** -23 < loss.max() < 2.0 ** -21 and loss[-1] > 0.97 * 2.0 ** -21


@pytest.mark.gpu
@pytest.mark.parametrize("which,shape", [("forward", BANDED), ("forward", ROUND), ("backward_input", CIRCLE), ("backward_input", GAPS)])
def test_weights_near_the_end_of_the_exponent_range(which, shape):
    """include/scc.h: a weight of 2**-120 keeps an absolute error of up to 2**-126, which the other factor multiplies.  Every
    output within that, 2**-21 of its products' magnitudes and 2**-24 of them per rounding of at most 64 partial sums."""
    N, Cin, Cout, H, W, cg, co = shape
    gen = torch.Generator(device="cuda").manual_seed(9)
    x = torch.randn(N, Cin if which == "forward" else Cout, H, W, generator=gen, device="cuda") * 2.0 ** 40
    w = torch.randn(Cout, Cin // cg, generator=gen, device="cuda") * 2.0 ** -60 * 2.0 ** -60
    hx, hw = x.cpu().numpy(), w.cpu().numpy()
    run = (lambda a, b: O.forward(a, b, cg, co)) if which == "forward" else (lambda a, b: O.backward_input(a, b, Cin, cg, co))
    got = (S.scc_forward(x, w, cg, co) if which == "forward" else S.scc_backward_input(x, w, Cin, cg, co)).cpu().numpy()
    bound = run(np.abs(hx), (np.abs(hw) * (2.0 ** -21 + 64 * 2.0 ** -24) + 2.0 ** -126).astype(np.float32))
    assert np.all(np.abs(got - run(hx, hw)) <= bound)


@pytest.mark.gpu
@pytest.mark.parametrize("which,dtype,shape", [CASES[0], CASES[6], CASES[10], CASES[15]])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_non_finite_values_stay_in_their_column(which, dtype, shape, value):
    N, Cin, Cout, H, W, cg, co = shape
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    gen = torch.Generator(device="cuda").manual_seed(10)
    src = Cin if which == "forward" else Cout
    x = torch.randn(N, src, H, W, generator=gen, device="cuda").to(td)
    w = torch.randn(Cout, Cin // cg, generator=gen, device="cuda").to(td)
    call = (lambda: S.scc_forward(x, w, cg, co)) if which == "forward" else (lambda: S.scc_backward_input(x, w, Cin, cg, co))
    clean = call()
    x[N // 2, src // 2, H - 1, W - 1] = value            # the last pixel: where groups of columns overlap
    got = call()
    column = torch.zeros_like(got, dtype=torch.bool)
    column[N // 2, :, H - 1, W - 1] = True
    assert torch.equal(got[~column], clean[~column])
    hit = got[N // 2, :, H - 1, W - 1]
    if which == "forward":                               # every filter whose window has the channel
        L, step, _ = S.scc_window_params(Cin, Cout, cg, co)
        reads = (src // 2 - torch.arange(Cout, device="cuda") * step) % Cin < L
        assert not bool(torch.isfinite(hit[reads]).any())
    else:
        assert not bool(torch.isfinite(hit).all())


@pytest.mark.gpu
@pytest.mark.parametrize("which,dtype,shape", [CASES[0], CASES[7], CASES[10], CASES[15]])
def test_calls_with_a_workspace_in_a_graph(which, dtype, shape):
    """Every replay against the eager result, with other work and new inputs in between."""
    N, Cin, Cout, H, W, cg, co = shape
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    gen = torch.Generator(device="cuda").manual_seed(11)
    src, dst = (Cin, Cout) if which == "forward" else (Cout, Cin)
    query = S.scc_forward_workspace_bytes if which == "forward" else S.scc_backward_input_workspace_bytes
    x = torch.randn(N, src, H, W, generator=gen, device="cuda").to(td)
    w = torch.randn(Cout, Cin // cg, generator=gen, device="cuda").to(td)
    out, ws = torch.empty(N, dst, H, W, dtype=td, device="cuda"), torch.empty(query(*shape, td), dtype=torch.uint8, device="cuda")

    def call(**kw):
        return S.scc_forward(x, w, cg, co, **kw) if which == "forward" else S.scc_backward_input(x, w, Cin, cg, co, **kw)

    call(out=out, workspace=ws)                          # code objects are loaded before the capture
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(out=out, workspace=ws)
    for _ in range(3):
        x.copy_(torch.randn(x.shape, generator=gen, device="cuda"))
        w.copy_(torch.randn(w.shape, generator=gen, device="cuda"))
        out.fill_(float("nan"))
        ws.fill_(255)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, call())


@pytest.mark.parametrize("shape", [(4, 2048, 2048, 7, 7, 1, 0.5), (16, 768, 1533, 7, 7, 1, 0.5), (9, 880, 3520, 9, 9, 2, 0.5)])
def test_weights_that_outweigh_the_planes_are_not_packed(shape):
    assert [need(which, dtype, shape) for which in ("forward", "backward_input") for dtype in ("f32", "bf16")] == [0] * 4
