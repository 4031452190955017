"""Workspaces smaller than the query says.  Layers whose filters share many channels ask for more than they cannot do without:
scc_backward_weight and scc_backward run them on what the per-tile kernel needs (its partial sums, KS x Cout x L floats, nothing
where it is not split) and refuse less."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2101_00745_amd as S
import scc_workloads as Wk
from oracle import scc_oracle as O

FAKE = ctypes.c_void_p(0x1000)
# (N, Cin, Cout, H, W, cg, co, dtype), bytes both calls cannot do without; 0: NULL is accepted
LAYERS = [((20, 1024, 1024, 14, 14, 1, 0.5, 0), 0), ((16, 360, 870, 16, 16, 2, 0.33, 1), 0), ((24, 700, 1000, 7, 7, 1, 0.5, 1), 0),
          ((64, 512, 1024, 7, 7, 2, 0.33, 0), 3 * 1024 * 256 * 4), ((330, 120, 500, 11, 9, 2, 0.33, 0), 9 * 500 * 60 * 4),
          ((100, 104, 400, 23, 22, 1, 0.3, 1), 10 * 400 * 104 * 4), ((39, 64, 48, 5, 5, 2, 0.25, 0), 0),
          ((110, 640, 746, 3, 3, 8, 0.5, 1), 0)]


@pytest.mark.parametrize("shape,least", LAYERS)
def test_less_than_the_least_is_refused(shape, least):
    lib = S.load()
    assert lib.scc_backward_weight_workspace_bytes(*shape) >= least and lib.scc_backward_workspace_bytes(*shape) >= least
    if least:
        for ws, size in ((FAKE, least - 1), (None, 0), (ctypes.c_void_p(0x1010), least)):
            assert lib.scc_backward_weight(FAKE, FAKE, FAKE, *shape, ws, size, None) == -5
            assert lib.scc_backward(FAKE, FAKE, FAKE, FAKE, FAKE, *shape, ws, size, None) == -5


@pytest.mark.gpu
@pytest.mark.parametrize("shape,least", LAYERS)
def test_the_least_is_enough(shape, least):
    N, Cin, Cout, H, W, cg, co, code = shape
    layer = Wk.Layer("least", 9, N=N, Cin=Cin, Cout=Cout, H=H, W=W, cg=cg, co=co)
    td = torch.bfloat16 if code else torch.float32
    x, w, dy = (torch.from_numpy(a).to(td).cuda() for a in Wk.make_inputs(layer))
    hx, hw, hdy = (t.float().cpu().numpy() for t in (x, w, dy))
    ref_dx, ref_dw = O.backward_input(hdy, hw, Cin, cg, co), O.backward_weight(hx, hdy, cg, co)
    ws = torch.empty(least, dtype=torch.uint8, device="cuda") if least else None
    ws_ptr, st = ws.data_ptr() if least else None, torch.cuda.current_stream().cuda_stream
    dx, dw, dw1 = torch.empty_like(x), torch.empty(w.shape, device="cuda"), torch.empty(w.shape, device="cuda")
    lib = S.load()
    assert lib.scc_backward_weight(x.data_ptr(), dy.data_ptr(), dw1.data_ptr(), *shape, ws_ptr, least, st) == 0
    assert lib.scc_backward(x.data_ptr(), dy.data_ptr(), w.data_ptr(), dx.data_ptr(), dw.data_ptr(), *shape, ws_ptr, least, st) == 0
    for got, ref, bar in ((dw, ref_dw, 2e-5), (dw1, ref_dw, 2e-5), (dx, ref_dx, 1e-2 if code else 2e-5)):
        assert np.max(np.abs(got.float().cpu().numpy() - ref)) <= bar * np.max(np.abs(ref))


@pytest.mark.parametrize("shape,need", [((190, 800, 69, 16, 16, 8, 0.0, 1), 13 * 69 * 100 * 4), ((117, 416, 65, 28, 28, 8, 0.0, 1), 16 * 65 * 52 * 4)])
def test_scc_backward_asks_for_what_runs(shape, need):
    """Layers whose two passes share one grid never run scc_backward_weight's kernel, which alone would take more."""
    lib = S.load()
    assert lib.scc_backward_workspace_bytes(*shape) == need < lib.scc_backward_weight_workspace_bytes(*shape)
