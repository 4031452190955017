"""Depthwise stage and its gradients in bf16 on rows of whole quads, whose lanes move 16 bytes at stride 2: against binary64, on
rows of one quad and of several, on tensors aligned to 8 bytes only, and taps of the first and the last channel."""
import pytest
import torch

import paper_2101_00745_amd as S

# (N, C, Ho, Wo, stride): one strip of a plane; rows of 1, 2 and 3 quads; strips of 4, 2 and 1 rows; more than a wavefront's lanes; 3072
# workgroups for grad-input and one group of samples less, whose lanes write under four outputs and under two
LAYERS = [(1, 1, 4, 4, 2), (3, 5, 2, 4, 2), (2, 7, 5, 12, 2), (5, 9, 16, 16, 2), (33, 24, 8, 8, 2), (2, 7, 5, 12, 1), (33, 24, 8, 8, 1),
          (96, 128, 16, 16, 2), (95, 128, 16, 16, 2), (3073, 64, 4, 4, 2), (820, 64, 5, 12, 2), (512, 64, 2, 48, 2)]


@pytest.mark.gpu
@pytest.mark.parametrize("N,C,Ho,Wo,s", LAYERS)
@pytest.mark.parametrize("offset", [0, 4])
def test_against_binary64(N, C, Ho, Wo, s, offset):
    gen = torch.Generator(device="cuda").manual_seed(3)

    def tensor(*d):                                         # `offset` values behind an address that is aligned to 256 bytes
        t = torch.randn(torch.Size(d).numel() + offset, generator=gen, device="cuda").to(torch.bfloat16)
        return t[offset:].view(*d)
    x, k, dz = tensor(N, C, s * Ho, s * Wo), tensor(C, 3, 3), tensor(N, C, Ho, Wo)
    z = S.scc_depthwise3x3_forward(x, k, s)
    dx, dk = S.scc_depthwise3x3_backward(x, k, dz, s)
    alone, _ = S.scc_depthwise3x3_backward(x, k, dz, s, need_dk=False)
    xr, kr = (t.double().cpu().requires_grad_() for t in (x, k))
    zr = torch.nn.functional.conv2d(xr, kr[:, None], stride=s, padding=1, groups=C)
    zr.backward(dz.double().cpu())
    assert torch.equal(dx, alone)
    for got, want in ((z, zr.detach()), (dx, xr.grad)):
        # one rounding to bf16 is half of 2^-7 of the value; nine sums of up to 9 products of 6 in binary32 9 * 54 * 2^-24
        assert bool(((got.double().cpu() - want).abs() <= 2.0 ** -8 * want.abs() + 3e-5).all())
    assert float((dk.double().cpu() - kr.grad).abs().max()) <= 1e-5 * (N * Ho * Wo) ** 0.5 + 1e-6 * N * Ho * Wo
