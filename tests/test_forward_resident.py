"""The bf16 forward that keeps its weights in registers: which layers take it, and every element against the fp32 forward of the same
values (itself held to the oracle), with samples against the fp64 oracle."""
import numpy as np
import pytest
import torch

import paper_2101_00745_amd as S
from oracle import scc_oracle as O

RESIDENT = 3    # SCC_FORWARD_RESIDENT
LAYERS = [(128, 128, 512, 32, 32, 2, 0.33),      # a filter group's walk of 95 channels, some across channel 0
          (150, 128, 512, 31, 30, 2, 0.33),      # planes of 930 pixels: a sample's last columns overlap; tiles left over
          (703, 448, 448, 12, 12, 8, 0.33),      # walk of 182; windows on most channels, last filter group of 64 rows
          (1100, 56, 221, 12, 12, 1, 0.75),       # once around the circle of 56 channels; filters without number in the last group
          (363, 160, 317, 20, 20, 4, 0.33),      # walk of 103, 16 starts to a tile
          (592, 96, 144, 20, 18, 4, 0.75),       # two filter groups, the second of 16 rows
          (310, 192, 768, 12, 13, 4, 0.33)]      # rows of 312 bytes
EVEN = [(592, 96, 144, 20, 18, 4, 0.5), (274, 256, 1024, 14, 14, 4, 0.75), (370, 80, 160, 32, 32, 2, 0.0)]     # weights in whole fours: packed or this
OTHERS = [((258, 128, 512, 16, 16, 4, 0.5), 1), ((310, 192, 768, 12, 13, 4, 0.75), 1),      # one start to a tile
          ((712, 64, 256, 14, 14, 2, 0.25), 1), ((709, 128, 192, 12, 12, 8, 0.0), 1),
          ((626, 32, 125, 20, 20, 2, 0.75), 1), ((366, 32, 125, 28, 28, 4, 0.75), 1),       # four starts to a tile
          ((806, 64, 96, 16, 16, 8, 0.33), 1),                                              # windows of 8
          ((419, 96, 144, 28, 28, 2, 0.0), 2), ((486, 192, 288, 20, 20, 4, 0.33), 2),       # many columns of large planes
          ((18, 576, 2301, 32, 48, 8, 0.33), 2), ((235, 48, 96, 56, 56, 1, 0.33), 2), ((115, 448, 1792, 16, 16, 8, 0.0), 2)]


def path(layer, code, workspace=1 << 30):
    return S.load().scc_forward_path(*layer, code, workspace)


@pytest.mark.parametrize("layer", LAYERS)
def test_lines(layer):
    N, Cin, Cout, H, W, cg, co = layer
    assert path(layer, 1) == path(layer, 1, 0) == RESIDENT and path(layer, 0) != RESIDENT
    for other in ((N // 16, Cin, Cout, H, W, cg, co), (N, Cin, 40, H, W, cg, co), (N, Cin, Cout, 7, 7, cg, co)):      # few columns, few filters, odd planes
        assert path(other, 1) != RESIDENT
    assert path((N, Cin, Cout, H, W, 0, co), 1) == -2


def test_layers_that_are_faster_elsewhere():
    """Eligible, and slower here when x is still in the last level cache: 0.67 to 0.95 of the other kernel's speed."""
    for layer, other in OTHERS:
        assert path(layer, 1) == other and path(layer, 1, 0) == 1, layer
    for layer in EVEN:
        assert path(layer, 1) == RESIDENT and path(layer, 1, 0) == 1, layer


def test_outputs_end_before_the_offset_that_is_dropped():
    """Stores of rows without a filter go to byte 2**31 of y."""
    N, Cin, Cout, H, W, cg, co = LAYERS[0]
    last = (2**32 - 1) // (4 * Cout * H * W)
    assert path((last, Cin, Cout, H, W, cg, co), 1) == RESIDENT and last * Cout * H * W * 2 < 2**31
    assert path((last + 1, Cin, Cout, H, W, cg, co), 1) != RESIDENT


@pytest.mark.gpu
@pytest.mark.parametrize("layer", LAYERS)
def test_parity(layer):
    N, Cin, Cout, H, W, cg, co = layer
    gen = torch.Generator(device="cuda").manual_seed(21)
    x, w = (torch.randn(*d, generator=gen, device="cuda").bfloat16() for d in ((N, Cin, H, W), (Cout, Cin // cg)))
    y = torch.full((N, Cout, H, W), float("nan"), dtype=torch.bfloat16, device="cuda")
    S.scc_forward(x, w, cg, co, out=y)
    assert torch.equal(y, S.scc_forward(x, w, cg, co))          # with and without a workspace
    wide = S.scc_forward(x.float(), w.float(), cg, co)
    # bf16 keeps 8 bits, so half a unit of its last place is at most 2**-8 of a value; both sums are binary32
    bound = wide.abs() * 2.0 ** -8 + 2e-5 * float(wide.abs().max())
    assert bool(((y.float() - wide).abs() <= bound).all())
    some = torch.tensor([0, N // 3, N - 1], device="cuda")
    ref = O.forward(x[some].float().cpu().numpy(), w.float().cpu().numpy(), cg, co)
    assert np.max(np.abs(y[some].float().cpu().numpy() - ref)) <= 4e-3 * np.max(np.abs(ref))


@pytest.mark.gpu
@pytest.mark.parametrize("layer", EVEN)
def test_parity_of_even_weights(layer):
    """With a workspace here, without one in the per-tile kernel: the same definition."""
    N, Cin, Cout, H, W, cg, co = layer
    x, w, _ = inputs(layer, 26)
    wide = S.scc_forward(x.float(), w.float(), cg, co)
    bound = wide.abs() * 2.0 ** -8 + 2e-5 * float(wide.abs().max())          # as in test_parity
    for y in (S.scc_forward(x, w, cg, co), S.scc_forward(x, w, cg, co, out=torch.full_like(wide, float("nan"), dtype=torch.bfloat16))):
        assert bool(((y.float() - wide).abs() <= bound).all())


@pytest.mark.gpu
def test_an_output_on_odd_addresses_takes_another_kernel():
    N, Cin, Cout, H, W, cg, co = LAYERS[3]
    gen = torch.Generator(device="cuda").manual_seed(22)
    x, w = (torch.randn(*d, generator=gen, device="cuda").bfloat16() for d in ((N, Cin, H, W), (Cout, Cin // cg)))
    odd = torch.zeros(N * Cout * H * W + 1, dtype=torch.bfloat16, device="cuda")[1:].view(N, Cout, H, W)
    S.scc_forward(x, w, cg, co, out=odd)
    want = S.scc_forward(x, w, cg, co).float()                  # both rounded: a unit of the last place, 2**-7, apart at most
    assert bool(((odd.float() - want).abs() <= want.abs() * 2.0 ** -7 + 2e-5 * float(want.abs().max())).all())


def inputs(layer, seed):
    N, Cin, Cout, H, W, cg, co = layer
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return [torch.randn(*d, generator=gen, device="cuda").bfloat16() for d in ((N, Cin, H, W), (Cout, Cin // cg))] + [gen]


@pytest.mark.gpu
@pytest.mark.parametrize("layer", [LAYERS[1], LAYERS[2], LAYERS[3], LAYERS[5]])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_non_finite_values_stay_in_their_column(layer, value):
    """They reach every filter whose window has the channel, and may reach others at the same sample and pixel: a wavefront multiplies 96
    positions of the walk, those past a window by zero."""
    N, Cin, Cout, H, W, cg, co = layer
    x, w, _ = inputs(layer, 23)
    clean = S.scc_forward(x, w, cg, co)
    places = [(0, 0, 0, 0), (N // 2, Cin // 2, H - 1, W - 1), (N - 1, Cin - 1, H - 1, W - 2)]      # the last pixels: where groups of columns overlap
    column = torch.zeros(N, H, W, dtype=torch.bool, device="cuda")
    for n, c, h, v in places:
        x[n, c, h, v] = value
        column[n, h, v] = True
    got = S.scc_forward(x, w, cg, co)
    assert torch.equal(torch.where(column[:, None], 0, got), torch.where(column[:, None], 0, clean))
    L, step, _ = S.scc_window_params(Cin, Cout, cg, co)
    for n, c, h, v in places:
        reads = (c - torch.arange(Cout, device="cuda") * step) % Cin < L
        assert not bool(torch.isfinite(got[n, reads, h, v]).any())


@pytest.mark.gpu
@pytest.mark.parametrize("layer", LAYERS)
def test_nothing_is_written_outside_the_output(layer):
    """Rows without a filter are stored past the end of y, where the hardware drops them; a sample's last columns are stored twice."""
    N, Cin, Cout, H, W, cg, co = layer
    x, w, _ = inputs(layer, 24)
    size, guard = N * Cout * H * W, 1 << 20
    buf = torch.full((size + 2 * guard,), 3.0, dtype=torch.bfloat16, device="cuda")
    y = buf[guard:guard + size].view(N, Cout, H, W)
    S.scc_forward(x, w, cg, co, out=y)
    assert torch.equal(y, S.scc_forward(x, w, cg, co))
    assert bool((buf[:guard] == 3.0).all()) and bool((buf[guard + size:] == 3.0).all())


@pytest.mark.gpu
@pytest.mark.parametrize("layer", [LAYERS[1], LAYERS[3]])
def test_calls_in_a_graph(layer):
    """Every replay against the eager result, with other work and new inputs in between."""
    N, Cin, Cout, H, W, cg, co = layer
    x, w, gen = inputs(layer, 25)
    out = torch.empty(N, Cout, H, W, dtype=torch.bfloat16, device="cuda")
    S.scc_forward(x, w, cg, co, out=out)                        # code objects are loaded before the capture
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        S.scc_forward(x, w, cg, co, out=out)
    for _ in range(3):
        x.copy_(torch.randn(x.shape, generator=gen, device="cuda"))
        w.copy_(torch.randn(w.shape, generator=gen, device="cuda"))
        out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, S.scc_forward(x, w, cg, co))
