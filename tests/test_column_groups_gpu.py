"""Planes whose size is not a multiple of the 2 or 4 pixels a lane moves at once: the last group of a sample overlaps the
one before it, so forward and grad-input compute its first pixels twice and grad-weight has to count them once.  Every
remainder, in both data types, through every entry point, against the fp64 oracle with the suite's bars."""
import numpy as np
import pytest
import torch

import scc_workloads as Wk
from oracle import scc_oracle as O

pytestmark = pytest.mark.gpu

# (N, Cin, Cout, H, W, cg, co): planes of 1-11 pixels, 49 and 63; few and many columns (1, 2 or 4 columns per lane)
SHAPES = [(300, 32, 40, 1, 1, 2, 0.5), (150, 32, 40, 1, 2, 2, 0.5), (90, 32, 40, 3, 1, 2, 0.25), (70, 32, 40, 1, 5, 2, 0.5),
          (64, 64, 96, 1, 6, 1, 0.5), (60, 32, 40, 7, 1, 2, 0.33), (33, 64, 40, 3, 3, 2, 0.5), (31, 32, 40, 1, 11, 4, 0.0),
          (64, 256, 512, 7, 7, 2, 0.33), (40, 64, 64, 9, 7, 4, 0.5), (400, 64, 64, 9, 7, 1, 0.5)]


@pytest.mark.parametrize("dtype,tol", [(torch.float32, 2e-5), (torch.bfloat16, 1e-2)])
@pytest.mark.parametrize("shape", SHAPES)
def test_every_remainder(shape, dtype, tol):
    import paper_2101_00745_amd as S
    N, Cin, Cout, H, W, cg, co = shape
    layer = Wk.Layer("groups", 9, N=N, Cin=Cin, Cout=Cout, H=H, W=W, cg=cg, co=co)
    xd, wd, dyd = (torch.from_numpy(a).to(dtype).cuda() for a in Wk.make_inputs(layer))
    x, w, dy = (t.float().cpu().numpy() for t in (xd, wd, dyd))
    y = S.scc_forward(xd, wd, cg, co)
    dx = S.scc_backward_input(dyd, wd, Cin, cg, co)
    dw = S.scc_backward_weight(xd, dyd, cg, co)
    dx2, dw2 = S.scc_backward(xd, dyd, wd, cg, co)
    rdx, rdw = O.backward_input(dy, w, Cin, cg, co), O.backward_weight(x, dy, cg, co)
    for got, ref, bar in ((y, O.forward(x, w, cg, co), tol), (dx, rdx, tol), (dx2, rdx, tol), (dw, rdw, 2e-5), (dw2, rdw, 2e-5)):
        err = np.max(np.abs(got.float().cpu().numpy() - ref)) / np.max(np.abs(ref))
        assert err <= bar, (shape, dtype, err)


# planes that are no multiple of 4 pixels whose wide tiles would be shared by four wavefronts: pairs of columns, one, two and four
# wavefronts per tile; the last has too few pairs and keeps the wide tiles
THIN = [(64, 512, 1024, 7, 7, 2, 0.33), (9, 360, 1440, 14, 7, 1, 0.0), (38, 384, 576, 7, 7, 1, 0.5), (5, 512, 448, 5, 5, 1, 0.5)]


@pytest.mark.parametrize("dtype,tol", [(torch.float32, 2e-5), (torch.bfloat16, 1e-2)])
@pytest.mark.parametrize("shape", THIN)
def test_forward_of_thin_layers_without_workspace(shape, dtype, tol):
    import paper_2101_00745_amd as S
    N, Cin, Cout, H, W, cg, co = shape
    layer = Wk.Layer("thin", 9, N=N, Cin=Cin, Cout=Cout, H=H, W=W, cg=cg, co=co)
    xd, wd, _ = (torch.from_numpy(a).to(dtype).cuda() for a in Wk.make_inputs(layer))
    out = torch.full((N, Cout, H, W), float("nan"), dtype=dtype, device="cuda")
    S.scc_forward(xd, wd, cg, co, out=out)
    ref = O.forward(xd.float().cpu().numpy(), wd.float().cpu().numpy(), cg, co)
    assert np.max(np.abs(out.float().cpu().numpy() - ref)) <= tol * np.max(np.abs(ref))
