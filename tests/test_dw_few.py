"""The DW + SCC forward for layers with few columns: one kernel on maps of rows of 4 or of 2x2 pixels."""
import numpy as np
import pytest
import torch

import paper_2101_00745_amd as S
from oracle import scc_oracle as O

# (N, Cin, Cout, Ho, Wo, stride, cg, co): one image (fewer columns than a tile), column counts below, at and above tiles of 32, 64 and
# 128, one / two / four column groups per workgroup (spans from 64 to 1024 channels), one and two filter tiles per workgroup, partial
# tiles of filters, windows that start off the groups of 16 channels and wrap, rows of 4 on maps that are not square
CASES = [(1, 64, 40, 4, 4, 1, 2, 0.5), (1, 512, 512, 4, 4, 1, 2, 0.5), (1, 512, 96, 2, 2, 2, 2, 0.5), (9, 1024, 200, 2, 2, 1, 2, 0.5),
         (2, 256, 33, 4, 4, 2, 1, 0.0), (3, 256, 64, 4, 4, 1, 4, 0.25), (7, 176, 61, 5, 4, 1, 2, 0.5), (5, 80, 90, 1, 4, 2, 1, 0.75),
         (12, 240, 130, 3, 4, 2, 4, 0.4), (33, 64, 128, 2, 2, 1, 1, 0.5), (128, 512, 512, 4, 4, 1, 2, 0.5), (110, 512, 500, 4, 4, 1, 2, 0.5),
         (70, 256, 768, 4, 4, 2, 2, 0.5), (6, 1600, 64, 4, 4, 1, 2, 0.5), (40, 128, 128, 2, 2, 2, 8, 0.5), (8, 96, 24, 4, 4, 1, 3, 1.0),
         # eight wavefronts: spans of 272 to 1024 channels, the last wavefronts with little or nothing of them
         (16, 1024, 1024, 2, 2, 1, 2, 0.5), (3, 272, 70, 4, 4, 2, 1, 0.5), (2, 528, 48, 2, 2, 2, 1, 0.5), (5, 304, 96, 5, 4, 1, 1, 0.25),
         # on both sides of the lines to the two stages: workgroups' number, rounds of a wavefront, width of a workgroup
         (16, 256, 1024, 4, 4, 2, 2, 0.5), (17, 256, 1024, 4, 4, 2, 2, 0.5), (16, 512, 64, 4, 4, 1, 1, 0.5), (66, 512, 96, 4, 4, 1, 1, 0.5),
         (30, 144, 576, 2, 2, 1, 1, 0.0), (26, 256, 300, 2, 2, 2, 2, 0.25)]


def tensors(case, dtype, shift=0):
    N, Cin, Cout, Ho, Wo, s, cg, co = case
    gen = torch.Generator().manual_seed(11)
    out = []
    for d in ((N, Cin, Ho * s, Wo * s), (Cin, 3, 3), (Cout, Cin // cg)):
        n = int(np.prod(d))
        t = torch.empty(n + shift, dtype=dtype, device="cuda")[shift:]       # shift: not aligned to 16 bytes
        t.copy_(torch.randn(n, generator=gen).to(dtype))
        out.append(t.view(d))
    return out


@pytest.mark.gpu
@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("case", CASES)
def test_against_the_oracle(case, dtype, shift):
    N, Cin, Cout, Ho, Wo, s, cg, co = case
    x, k, w = tensors(case, dtype, shift)
    y = S.scc_dw_forward(x, k, w, cg, co, s)
    ref = O.depthwise_scc_forward(*(t.float().cpu().numpy() for t in (x, k, w)), cg, co, s)
    # bf16: the depthwise output and the result are rounded to 2^-9 of themselves at most
    bar = 2e-5 if dtype == torch.float32 else 1e-2
    assert np.max(np.abs(y.float().cpu().numpy() - ref)) <= bar * np.max(np.abs(ref))
    assert torch.equal(y, S.scc_dw_forward(x, k, w, cg, co, s))                # fixed order of the sums
    if dtype == torch.float32:
        two = S.scc_dw_forward(x, k, w, cg, co, s, fused=False)
        err = [float((t.double().cpu() - torch.from_numpy(np.asarray(ref, dtype=np.float64))).norm()) for t in (y, two)]
        assert err[0] <= 1.1 * err[1]                                          # no further from binary64 than the two stages


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_a_given_workspace_holds_the_depthwise_output(dtype):
    case = (16, 512, 512, 4, 4, 1, 2, 0.5)
    N, Cin, Cout, Ho, Wo, s, cg, co = case
    x, k, w = tensors(case, dtype)
    need = S.scc_dw_forward_workspace_bytes(N, Cin, Cout, Ho * s, Wo * s, s, cg, co, dtype)
    assert need == N * Cin * Ho * Wo * x.element_size()
    ws = torch.zeros(need, dtype=torch.uint8, device="cuda")
    y = S.scc_dw_forward(x, k, w, cg, co, s, workspace=ws)
    z = S.scc_depthwise3x3_forward(x, k, s)
    assert torch.equal(ws.view(dtype).view(z.shape), z)
    assert torch.equal(y, S.scc_dw_forward(x, k, w, cg, co, s, fused=False))
    # binary32 sums in another order; bf16 results rounded to 2^-9 of themselves
    own = S.scc_dw_forward(x, k, w, cg, co, s, out=torch.empty_like(y))
    assert torch.equal(own, S.scc_dw_forward(x, k, w, cg, co, s))                # one kernel, with and without an out tensor
    assert (own.float() - y.float()).abs().max() <= (2e-5 if dtype == torch.float32 else 1e-2) * y.float().abs().max()
