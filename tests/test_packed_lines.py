"""Which forward takes packed weights on layers of whole groups of 4 pixels and weights and one window per tile."""
import numpy as np
import pytest
import torch

import paper_2101_00745_amd as S
from oracle import scc_oracle as O

# (N, Cin, Cout, H, W, cg, co), dtype, packed
LINES = [
    # long walks whose planes the shared forward shares between nearly four tiles are left to it, shorter ones and those shared less are not
    ((141, 800, 800, 12, 12, 4, 0.5), torch.float32, False), ((16, 960, 3840, 16, 16, 4, 0.0), torch.float32, False),
    ((157, 272, 272, 20, 20, 1, 0.5), torch.float32, True), ((122, 320, 1280, 16, 24, 4, 0.5), torch.float32, True),
    ((128, 256, 256, 16, 16, 1, 0.5), torch.float32, True),
    # rows that do not fill their groups are taken from three fetches on, rows that do from seven
    ((47, 688, 344, 14, 14, 1, 0.5), torch.bfloat16, True), ((51, 360, 360, 16, 16, 1, 0.5), torch.bfloat16, True),
    ((446, 544, 2176, 4, 4, 4, 0.5), torch.bfloat16, False), ((128, 256, 256, 16, 16, 1, 0.5), torch.bfloat16, True)]


@pytest.mark.parametrize("layer,dtype,packed", LINES)
def test_lines(layer, dtype, packed):
    N, Cin, Cout, H, W, cg, co = layer
    assert (S.scc_forward_workspace_bytes(N, Cin, Cout, H, W, cg, co, dtype) > 0) == packed


@pytest.mark.gpu
@pytest.mark.parametrize("layer,dtype,packed", [c for c in LINES if c[0][0] in (47, 51, 141)])
def test_layers_that_changed_sides(layer, dtype, packed):
    N, Cin, Cout, H, W, cg, co = layer
    gen = torch.Generator(device="cuda").manual_seed(14)
    x, w = (torch.randn(*d, generator=gen, device="cuda").to(dtype) for d in ((N, Cin, H, W), (Cout, Cin // cg)))
    y = S.scc_forward(x, w, cg, co)[:2]
    ref = O.forward(x[:2].float().cpu().numpy(), w.float().cpu().numpy(), cg, co)
    bar = 2e-6 if dtype == torch.float32 else 4e-3          # binary32 sums; half a unit of bf16's last place is 2^-9 of a value
    assert np.max(np.abs(y.float().cpu().numpy().astype(np.float64) - ref)) <= bar * np.max(np.abs(ref))
