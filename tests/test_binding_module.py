"""The native part of the binding is the plain calls' shorter way, not a condition: without it every call takes the general way through
ctypes, on the same kernels."""
import os
import sys
import types

import pytest
import torch

import paper_2101_00745_amd as S
from paper_2101_00745_amd import build
from paper_2101_00745_amd import scc as B


@pytest.fixture
def absent(monkeypatch):
    """A package whose native part cannot be imported."""
    monkeypatch.setitem(sys.modules, "paper_2101_00745_amd._binding", None)
    monkeypatch.delattr("paper_2101_00745_amd._binding", raising=False)
    monkeypatch.setattr(B, "_native", None)


def calls(x, k, w, dy):
    return (lambda: S.scc_forward(x, w, 2, 0.5), lambda: S.scc_backward(x, dy, w, 2, 0.5), lambda: S.scc_dw_forward(x, k, w, 2, 0.5),
            lambda: S.scc_dw_backward(x, k, w, dy, 2, 0.5))


@pytest.mark.filterwarnings("ignore:plain calls")
def test_calls_reach_the_general_way(absent):
    x = torch.zeros(1, 8, 4, 4)
    for c in calls(x, torch.zeros(8, 3, 3), torch.zeros(8, 4), x):
        with pytest.raises(ValueError, match="must live on the GPU"):
            c()


def test_the_absence_is_reported_once(absent):
    with pytest.warns(RuntimeWarning, match="plain calls"):
        B._load_native()
    assert B._native is not None and B._native.forward(None) is None


@pytest.mark.gpu
@pytest.mark.filterwarnings("ignore:plain calls")
def test_results_are_the_same(absent, monkeypatch):
    gen = torch.Generator(device="cuda").manual_seed(4)
    args = [torch.randn(*d, generator=gen, device="cuda") for d in ((3, 32, 6, 4), (32, 3, 3), (24, 16), (3, 24, 6, 4))]
    without = [c() for c in calls(*args)]
    monkeypatch.undo()
    for a, b in zip(without, [c() for c in calls(*args)]):
        for s, t in zip(a if isinstance(a, tuple) else (a,), b if isinstance(b, tuple) else (b,)):
            assert torch.equal(s, t)


def never(*args):
    raise AssertionError("called into a module of another torch")


@pytest.mark.parametrize("built_for", [None, "cpython-310 torch 2.4.0 0000"])
def test_a_module_of_another_torch_is_not_called(absent, monkeypatch, built_for):
    other = types.ModuleType("paper_2101_00745_amd._binding")
    other.forward = other.backward = other.dw_forward = other.dw_backward = never
    if built_for:
        other.built_for = built_for
    monkeypatch.setitem(sys.modules, other.__name__, other)
    with pytest.warns(RuntimeWarning, match="not built for this torch"):
        with pytest.raises(ValueError, match="must live on the GPU"):
            S.scc_forward(torch.zeros(1, 8, 4, 4), torch.zeros(8, 4), 2, 0.5)


def test_the_built_module_is_for_this_torch(monkeypatch):
    B.load()
    from paper_2101_00745_amd import _binding
    assert _binding.built_for == build.binding_tag() and os.path.samefile(_binding.__file__, build.BINDING_LIB)
    monkeypatch.setattr(build, "binding_tag", lambda: "cpython-310 torch 2.4.0 0000")
    assert build.stale()                                     # built again where torch changed


@pytest.mark.parametrize("hipcc", ["hipcc", "/opt/rocm/bin/hipcc"])
def test_the_headers_of_a_compiler_named_by_command(monkeypatch, hipcc):
    """HIPCC may be a path or a name on PATH; the ROCm headers are those beside it either way."""
    monkeypatch.setattr(build, "HIPCC", hipcc)
    monkeypatch.setenv("PATH", "/opt/rocm/bin" + os.pathsep + os.environ["PATH"])
    seen = []
    monkeypatch.setattr(build, "_run", lambda cmd, verbose: seen.extend(cmd))
    monkeypatch.setattr(build.os, "replace", lambda a, b: None)
    build.build_binding()
    assert any(c.startswith("-I") and os.path.exists(os.path.join(c[2:], "hip", "hip_runtime_api.h")) for c in seen)
