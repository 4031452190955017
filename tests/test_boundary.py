"""Host-side tests of the C ABI: the library loads, exports what include/scc.h declares,
and rejects bad arguments on the host (no GPU is touched by any call made here)."""
import ctypes
import math
import os
import re

import pytest

import paper_2101_00745_amd as S
from paper_2101_00745_amd import scc as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
FAKE = ctypes.c_void_p(0x1000)  # non-NULL, never dereferenced: every call below fails validation first


def declared_functions():
    text = open(os.path.join(ROOT, "include", "scc.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(scc_[a-z0-9_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    lib = S.load()
    names = declared_functions()
    assert sorted(names) == sorted(B.SYMBOLS)
    for name in names:
        assert getattr(lib, name) is not None


def test_status_strings():
    for code in range(0, -8, -1):
        s = S.scc_status_string(code)
        assert s.startswith("SCC_")
    assert "unknown" in S.scc_status_string(-99)


def alg1_period(Cin, Cout, cg, co):
    """Distinct window starts among the first Cout filters (Algorithm 1: filter k starts k * (gw - ov) channels on, folded)."""
    gw = Cin // cg
    return len({(k * (gw - int(co * gw))) % Cin for k in range(Cout)})


@pytest.mark.parametrize("Cin,Cout,cg,co", [(4, 4, 2, 0.5), (256, 256, 4, 0.0), (256, 256, 4, 0.25), (256, 256, 4, 0.5),
                                            (256, 256, 4, 0.75), (512, 512, 8, 0.5), (128, 512, 2, 0.33),
                                            (6, 9, 2, 1 / 3), (16, 5, 1, 0.0), (16, 5, 1, 1.0), (16, 3, 2, 0.25),
                                            (100, 77, 1, 0.29), (1024, 1024, 2, 0.5)])
def test_window_params(Cin, Cout, cg, co):
    L, stride, period = S.scc_window_params(Cin, Cout, cg, co)
    assert L == Cin // cg
    assert stride == L - int(co * L)
    assert period == alg1_period(Cin, Cout, cg, co)


def test_window_params_paper_values():
    # Section 5.4: Cin=4, co=50% (cg=2) -> cyclic distance 4; Section 4.2: cg=2/co=50% -> 4 for any Cin
    assert S.scc_window_params(4, 8, 2, 0.5)[2] == 4
    assert S.scc_window_params(512, 512, 2, 0.5)[2] == 4
    assert S.scc_window_params(64, 128, 2, 0.5)[0] == 32


BAD = [
    (dict(N=0), B.SccError, -2), (dict(Cin=-4), B.SccError, -2), (dict(Cout=0), B.SccError, -2),
    (dict(H=0), B.SccError, -2), (dict(W=-1), B.SccError, -2), (dict(cg=0), B.SccError, -2),
    (dict(cg=3), B.SccError, -2),                      # 8 % 3 != 0
    (dict(co=-0.01), B.SccError, -3), (dict(co=1.01), B.SccError, -3), (dict(co=math.nan), B.SccError, -3),
    (dict(co=math.inf), B.SccError, -3), (dict(dtype=2), B.SccError, -4), (dict(dtype=-1), B.SccError, -4),
    (dict(N=1 << 20, H=1 << 10, W=1 << 10), B.SccError, -2),   # N*H*W overflows 32-bit columns
]


def _call(which, **over):
    a = dict(N=2, Cin=8, Cout=6, H=3, W=3, cg=2, co=0.5, dtype=0)
    a.update(over)
    lib = S.load()
    shape = (a["N"], a["Cin"], a["Cout"], a["H"], a["W"], a["cg"], a["co"], a["dtype"])
    if which == "fwd":
        return lib.scc_forward(FAKE, FAKE, FAKE, *shape, None)
    if which == "bwi":
        return lib.scc_backward_input(FAKE, FAKE, FAKE, *shape, None)
    if which == "bwd":
        return lib.scc_backward(FAKE, FAKE, FAKE, FAKE, FAKE, *shape, None, 0, None)
    if which == "bww_static":
        return lib.scc_backward_weight_static(FAKE, FAKE, FAKE, *shape, None)
    return lib.scc_backward_weight(FAKE, FAKE, FAKE, *shape, None, 0, None)


@pytest.mark.parametrize("which", ["fwd", "bwi", "bww", "bwd", "bww_static"])
@pytest.mark.parametrize("over,exc,code", BAD)
def test_invalid_arguments_are_rejected_on_the_host(which, over, exc, code):
    assert _call(which, **over) == code
    shape = dict(N=2, Cin=8, Cout=6, H=3, W=3, cg=2, co=0.5, dtype=0)
    shape.update(over)
    args = [shape[k] for k in ("N", "Cin", "Cout", "H", "W", "cg", "co", "dtype")]
    assert S.load().scc_backward_weight_workspace_bytes(*args) == 0
    assert S.load().scc_backward_workspace_bytes(*args) == 0


def test_null_pointers_are_rejected():
    lib = S.load()
    shape = (2, 8, 6, 3, 3, 2, 0.5, 0)
    for i in range(3):
        ptrs = [FAKE, FAKE, FAKE]
        ptrs[i] = None
        assert lib.scc_forward(*ptrs, *shape, None) == -1
        assert lib.scc_backward_input(*ptrs, *shape, None) == -1
        assert lib.scc_backward_weight(*ptrs, *shape, None, 0, None) == -1
        assert lib.scc_backward_weight_static(*ptrs, *shape, None) == -1
    for i in range(5):
        ptrs = [FAKE] * 5
        ptrs[i] = None
        assert lib.scc_backward(*ptrs, *shape, None, 0, None) == -1


DW_BAD = [
    (dict(N=0), -2), (dict(Cin=-4), -2), (dict(Cout=0), -2), (dict(H=0), -2), (dict(W=-1), -2), (dict(cg=0), -2),
    (dict(cg=3), -2), (dict(s=0), -2), (dict(s=-2), -2), (dict(co=-0.01), -3), (dict(co=math.nan), -3),
    (dict(dtype=2), -4), (dict(N=1 << 20, H=1 << 10, W=1 << 10), -2),
]


@pytest.mark.parametrize("over,code", DW_BAD)
def test_dw_block_invalid_arguments_are_rejected_on_the_host(over, code):
    a = dict(N=2, Cin=8, Cout=6, H=5, W=5, s=1, cg=2, co=0.5, dtype=0)
    a.update(over)
    lib = S.load()
    shape = (a["N"], a["Cin"], a["Cout"], a["H"], a["W"], a["s"], a["cg"], a["co"], a["dtype"])
    assert lib.scc_dw_forward(FAKE, FAKE, FAKE, FAKE, *shape, FAKE, 1 << 30, None) == code
    assert lib.scc_dw_forward_workspace_bytes(*shape) == 0
    if not ({"Cout", "cg", "co"} & set(over)):
        assert lib.scc_depthwise3x3_forward(FAKE, FAKE, FAKE, a["N"], a["Cin"], a["H"], a["W"], a["s"], a["dtype"],
                                            None) == code


def test_dw_block_null_pointers_and_workspace():
    lib = S.load()
    shape = (2, 8, 6, 5, 5, 2, 2, 0.5, 0)       # Cin = 8 is not a multiple of 16: the two-stage path, needs a workspace
    need = lib.scc_dw_forward_workspace_bytes(*shape)
    assert need == 2 * 8 * 3 * 3 * 4            # the depthwise output: N x Cin x 3 x 3 binary32 values
    for i in range(4):
        ptrs = [FAKE] * 4
        ptrs[i] = None
        assert lib.scc_dw_forward(*ptrs, *shape, FAKE, need, None) == -1
    assert lib.scc_dw_forward(FAKE, FAKE, FAKE, FAKE, *shape, None, 0, None) == -5
    assert lib.scc_dw_forward(FAKE, FAKE, FAKE, FAKE, *shape, FAKE, need - 1, None) == -5
    assert lib.scc_dw_forward(FAKE, FAKE, FAKE, FAKE, *shape, ctypes.c_void_p(0x1010), need, None) == -5   # misaligned
    for i in range(3):
        ptrs = [FAKE] * 3
        ptrs[i] = None
        assert lib.scc_depthwise3x3_forward(*ptrs, 2, 8, 5, 5, 1, 0, None) == -1
    # layers the fused kernel takes need no workspace
    assert lib.scc_dw_forward_workspace_bytes(128, 256, 256, 16, 16, 1, 4, 0.5, 0) == 0
    assert lib.scc_dw_forward_workspace_bytes(128, 256, 256, 16, 16, 1, 4, 0.5, 1) == 128 * 256 * 256 * 2   # bf16
    # a layer the fused kernel can run but that is faster in two stages: a workspace is asked for, and the query says
    # that a call without one is served by the fused kernel
    deep = (128, 512, 512, 4, 4, 1, 2, 0.5, 0)
    assert lib.scc_dw_forward_workspace_bytes(*deep) == 128 * 512 * 16 * 4 and lib.scc_dw_forward_fusable(*deep) == 1
    assert lib.scc_dw_forward_fusable(*shape) == 0 and lib.scc_dw_forward_fusable(128, 256, 256, 16, 16, 1, 4, 0.5, 1) == 0
    assert lib.scc_dw_forward_fusable(128, 256, 256, 16, 16, 0, 4, 0.5, 0) == -2
    assert lib.scc_dw_forward_fusable(128, 256, 256, 16, 16, 1, 4, 0.5, 7) == -4
    # the depthwise stage's gradients: dz is required, at least one output, and the input each output needs
    args = (2, 8, 5, 5, 1, 0)
    need = lib.scc_depthwise3x3_backward_workspace_bytes(*args)
    assert need == 2 * 8 * 9 * 4                  # two slices of the batch x 8 channels x 9 taps
    assert lib.scc_depthwise3x3_backward(FAKE, FAKE, None, FAKE, FAKE, *args, FAKE, need, None) == -1
    assert lib.scc_depthwise3x3_backward(FAKE, FAKE, FAKE, None, None, *args, FAKE, need, None) == -1
    assert lib.scc_depthwise3x3_backward(None, FAKE, FAKE, FAKE, FAKE, *args, FAKE, need, None) == -1    # dkdw needs x
    assert lib.scc_depthwise3x3_backward(FAKE, None, FAKE, FAKE, FAKE, *args, FAKE, need, None) == -1    # dx needs kdw
    assert lib.scc_depthwise3x3_backward(FAKE, FAKE, FAKE, FAKE, FAKE, *args, None, 0, None) == -5
    assert lib.scc_depthwise3x3_backward(FAKE, FAKE, FAKE, FAKE, FAKE, *args, FAKE, need - 1, None) == -5
    assert lib.scc_depthwise3x3_backward(FAKE, FAKE, FAKE, FAKE, FAKE, 2, 8, 5, 5, 0, 0, FAKE, need, None) == -2
    assert lib.scc_depthwise3x3_backward(FAKE, FAKE, FAKE, FAKE, FAKE, 2, 8, 5, 5, 1, 3, FAKE, need, None) == -4
    assert lib.scc_depthwise3x3_backward_workspace_bytes(0, 8, 5, 5, 1, 0) == 0
    assert lib.scc_depthwise3x3_out(32, 2) == 16 and lib.scc_depthwise3x3_out(7, 2) == 4
    assert lib.scc_depthwise3x3_out(0, 1) == -2 and lib.scc_depthwise3x3_out(5, 0) == -2


def test_backward_workspace_is_checked_on_the_host():
    # a layer the fused backward kernel takes: it needs K-split scratch, and a call without it is refused
    lib = S.load()
    shape = (64, 256, 256, 16, 16, 4, 0.5, 0)
    need = lib.scc_backward_workspace_bytes(*shape)
    assert need > 0 and need >= lib.scc_backward_weight_workspace_bytes(*shape)
    assert lib.scc_backward(FAKE, FAKE, FAKE, FAKE, FAKE, *shape, None, 0, None) == -5
    assert lib.scc_backward(FAKE, FAKE, FAKE, FAKE, FAKE, *shape, FAKE, need - 1, None) == -5
    assert lib.scc_backward(FAKE, FAKE, FAKE, FAKE, FAKE, *shape, ctypes.c_void_p(0x1004), need, None) == -5


def test_binding_refuses_cpu_tensors():
    import torch
    x = torch.zeros(1, 4, 2, 2)
    w = torch.zeros(4, 2)
    with pytest.raises(ValueError):
        S.scc_forward(x, w, 2, 0.5)
    with pytest.raises(ValueError):
        S.scc_backward_input(x, w, 4, 2, 0.5)
    with pytest.raises(ValueError):
        S.scc_backward_weight(x, x, 2, 0.5)


def test_package_imports_on_a_torch_without_the_raw_stream_function():
    """The function is not part of torch's public interface; host-only calls need no stream at all."""
    import subprocess
    import sys
    code = ("import torch\n"
            "if hasattr(torch._C, '_cuda_getCurrentRawStream'): del torch._C._cuda_getCurrentRawStream\n"
            "import paper_2101_00745_amd as S\n"
            "assert S.scc_window_params(4, 4, 2, 0.5) == (2, 1, 4) and S.scc._raw_stream is S.scc._stream_address\n")
    subprocess.run([sys.executable, "-c", code], cwd=ROOT, check=True, timeout=300)


@pytest.mark.gpu
def test_both_ways_to_the_stream_agree():
    import torch
    for stream in (torch.cuda.default_stream(), torch.cuda.Stream()):
        with torch.cuda.stream(stream):
            index = torch.cuda.current_device()
            assert B._raw_stream(index) == B._stream_address(index) == stream.cuda_stream
