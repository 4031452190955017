"""Forward and grad-input with one address per chunk of planes (layers whose chunks stay inside the channel circle, window starts with
a multiple of 8 filters) and the layers beside them that take an address per plane."""
import numpy as np
import pytest
import torch

import paper_2101_00745_amd as S
from oracle import scc_oracle as O

# (N, Cin, Cout, H, W, cg, co): 8, 16 and 24 filters per window start and one filter more or less; an odd number of chunks per block;
# windows that wrap; Cin and starts that are multiples of 8, of 4 and neither; tiles with missing filters, channels and columns;
# 64, 65 and 2000 columns; one, two and four wavefronts per tile
LAYERS = [(4, 64, 64, 4, 4, 4, 0.5), (5, 64, 65, 4, 4, 4, 0.5), (3, 96, 48, 8, 8, 2, 0.5), (3, 96, 47, 8, 8, 2, 0.5), (13, 48, 72, 5, 1, 3, 0.5),
          (2, 40, 40, 10, 10, 1, 0.2), (2, 36, 72, 9, 7, 1, 0.25), (3, 52, 104, 6, 6, 2, 0.5), (3, 30, 24, 8, 8, 2, 0.33), (1, 1024, 512, 8, 8, 2, 0.5),
          (8, 256, 256, 5, 5, 8, 0.25), (20, 256, 128, 10, 10, 4, 0.25), (1, 512, 96, 9, 9, 1, 0.0), (40, 72, 144, 7, 7, 3, 0.5)]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("layer", LAYERS)
def test_against_the_oracle(layer, dtype):
    N, Cin, Cout, H, W, cg, co = layer
    gen = torch.Generator(device="cuda").manual_seed(7)
    x, w, dy = (torch.randn(*d, generator=gen, device="cuda").to(dtype) for d in ((N, Cin, H, W), (Cout, Cin // cg), (N, Cout, H, W)))
    xh, wh, gh = (t.float().cpu().numpy() for t in (x, w, dy))
    bar = 2e-6 if dtype == torch.float32 else 4e-3          # binary32 sums; half a unit of bf16's last place is 2^-9 of a value
    for got, ref in ((S.scc_forward(x, w, cg, co, out=torch.empty_like(dy)), O.forward(xh, wh, cg, co)),
                     (S.scc_backward_input(dy, w, Cin, cg, co, out=torch.empty_like(x)), O.backward_input(gh, wh, Cin, cg, co)),
                     (S.scc_backward(x, dy, w, cg, co)[0], O.backward_input(gh, wh, Cin, cg, co))):
        err = np.abs(got.float().cpu().numpy().astype(np.float64) - ref)
        assert np.max(err) <= bar * np.max(np.abs(ref))
