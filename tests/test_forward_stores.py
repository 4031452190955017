"""Forward: rows written past the caches (planes of whole 64-byte pieces) and through them, by whole tiles of filters and columns and
by partial ones."""
import numpy as np
import pytest
import torch

import paper_2101_00745_amd as S
from oracle import scc_oracle as O


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("N,H,W", [(64, 2, 2), (33, 4, 4), (16, 4, 8), (40, 5, 5), (128, 8, 4), (21, 7, 7), (3, 16, 16), (2, 12, 6)])
@pytest.mark.parametrize("Cin,Cout,cg", [(64, 64, 2), (64, 61, 8)])
def test_planes_of_whole_and_broken_pieces(Cin, Cout, cg, N, H, W, dtype):
    gen = torch.Generator(device="cuda").manual_seed(12)
    x, w = (torch.randn(*d, generator=gen, device="cuda").to(dtype) for d in ((N, Cin, H, W), (Cout, Cin // cg)))
    y = torch.full((N + 2, Cout, H, W), 7.0, dtype=dtype, device="cuda")     # a sample before and behind: nothing outside is written
    S.scc_forward(x, w, cg, 0.5, out=y[1:-1])
    ref = O.forward(x.float().cpu().numpy(), w.float().cpu().numpy(), cg, 0.5)
    bar = 2e-6 if dtype == torch.float32 else 4e-3          # binary32 sums; half a unit of bf16's last place is 2^-9 of a value
    assert np.max(np.abs(y[1:-1].float().cpu().numpy().astype(np.float64) - ref)) <= bar * np.max(np.abs(ref))
    assert bool((y[0] == 7).all()) and bool((y[-1] == 7).all())


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("Cin,cg", [(1, 1), (2, 1), (3, 1), (8, 2), (10, 2), (7, 1), (33, 3), (192, 2)])
def test_any_shape(Cin, cg, dtype):
    """Fewer columns than the tiled kernels take; windows of whole and partial rounds of four channels, wrapping."""
    gen = torch.Generator(device="cuda").manual_seed(13)
    x, w = (torch.randn(*d, generator=gen, device="cuda").to(dtype) for d in ((3, Cin, 4, 5), (19, Cin // cg)))
    ref = O.forward(x.float().cpu().numpy(), w.float().cpu().numpy(), cg, 0.5)
    bar = 2e-6 if dtype == torch.float32 else 4e-3
    assert np.max(np.abs(S.scc_forward(x, w, cg, 0.5).float().cpu().numpy().astype(np.float64) - ref)) <= bar * np.max(np.abs(ref))
