"""Grids of several generations, dealt to the XCDs in runs of 16 column tiles (scc_common.h, Deal): every element is written,
and samples of the first and last runs and of the part that is left over agree with the fp64 oracle."""
import numpy as np
import pytest
import torch

import paper_2101_00745_amd as S
from oracle import scc_oracle as O

# N, Cin, Cout, H, W, cg, co: tiles of 128 columns, groups per tile
LAYERS = [(256, 64, 256, 16, 16, 1, 0.5),      # 512 x 2: whole runs only
          (259, 64, 256, 16, 16, 2, 0.5),      # 518 x 2: six tiles left over
          (301, 64, 384, 13, 9, 4, 0.25),      # planes of 117: tiles that share samples, three groups
          (66, 32, 256, 32, 32, 2, 0.33),      # banded windows: packed weights in bf16 and fp32
          (255, 256, 64, 16, 16, 2, 0.5)]      # grad-input: two groups of channel blocks, the last run not whole


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("layer", LAYERS)
def test_every_tile_once(layer, dtype):
    N, Cin, Cout, H, W, cg, co = layer
    gen = torch.Generator(device="cuda").manual_seed(3)
    x, dy, w = (torch.randn(*d, generator=gen, device="cuda").to(dtype)
                for d in ((N, Cin, H, W), (N, Cout, H, W), (Cout, Cin // cg)))
    y, dx = torch.full_like(dy, float("nan")), torch.full_like(x, float("nan"))
    S.scc_forward(x, w, cg, co, out=y)
    S.scc_backward_input(dy, w, Cin, cg, co, out=dx)
    assert bool(torch.isfinite(y).all()) and bool(torch.isfinite(dx).all())
    some = torch.tensor([0, 1, N // 8, N // 2, N - 2, N - 1], device="cuda")
    host = lambda t: t.float().cpu().numpy()
    bar = 2e-6 if dtype == torch.float32 else 4e-3          # binary32 sums; half a unit of bf16's last place is 2^-9 of a value
    for got, ref in ((y, O.forward(host(x[some]), host(w), cg, co)), (dx, O.backward_input(host(dy[some]), host(w), Cin, cg, co)),
                     (S.scc_forward(x, w, cg, co), O.forward(host(x[some]), host(w), cg, co))):
        assert np.max(np.abs(host(got[some]) - ref)) <= bar * np.max(np.abs(ref))
