"""Compile the HIP sources in csrc/ into libscc_hip.so (gfx950 only) and the Python binding's native part, in-tree."""
import glob
import os
import shutil
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
LIB = os.path.join(HERE, "libscc_hip.so")
MEMBW_SRC = os.path.join(CSRC, "membw", "membw.hip")
MEMBW_LIB = os.path.join(HERE, "libscc_membw.so")   # streaming kernels of the benchmark's copy ceiling; not the SCC ABI

BINDING_SRC = os.path.join(CSRC, "binding", "scc_binding.cpp")
# the Python binding's plain calls (host code against torch's C++ API, so for one interpreter and one torch: binding_tag)
BINDING_LIB = os.path.join(HERE, "_binding" + sysconfig.get_config_var("EXT_SUFFIX"))

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
COMPILE_FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-fno-gpu-rdc",
                 # packed fp32 VALU forms are kept out of the generated code on purpose
                 "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                 "-Wno-unused-command-line-argument", "-Wno-unknown-warning-option"]
LINK_FLAGS = ["--offload-arch=gfx950", "-fPIC", "-shared", "-fno-gpu-rdc", "-Wno-unused-command-line-argument"]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def rocm_root():
    """The ROCm tree that HIPCC, a path or a command name, belongs to."""
    hipcc = shutil.which(HIPCC)
    if hipcc is None:
        raise RuntimeError("no compiler %r (set HIPCC)" % HIPCC)
    return os.path.dirname(os.path.dirname(os.path.realpath(hipcc)))


def binding_tag():
    """What the native part of the binding is built for; it holds this text (`built_for`)."""
    import torch
    return "%s torch %s %s" % (sys.implementation.cache_tag, torch.__version__, torch.version.git_version)


def stale():
    if not os.path.exists(LIB) or not os.path.exists(BINDING_LIB):
        return True
    with open(BINDING_LIB, "rb") as f:
        if binding_tag().encode() not in f.read():
            return True
    t = min(os.path.getmtime(LIB), os.path.getmtime(BINDING_LIB))
    deps = sources() + [BINDING_SRC] + glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(INCLUDE, "*.h"))
    return any(os.path.getmtime(f) > t for f in deps)


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + res.stdout)
    if verbose and res.stdout.strip():
        print(res.stdout)


def build(force=True, verbose=False):
    """Build libscc_hip.so.  With force=False, only when a source is newer than the library.
    The translation units are compiled side by side (objects in a scratch directory), then linked."""
    if not force and not stale():
        return LIB
    import concurrent.futures
    import tempfile
    work = tempfile.mkdtemp(prefix="scc_build_")
    try:
        objs = []
        with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, len(sources()))) as pool:
            jobs = []
            for src in sources():
                obj = os.path.join(work, os.path.basename(src) + ".o")
                objs.append(obj)
                jobs.append(pool.submit(_run, [HIPCC] + COMPILE_FLAGS + ["-I", INCLUDE, "-I", CSRC, "-c", src, "-o", obj],
                                        verbose))
            for j in jobs:
                j.result()
        tmp = LIB + ".tmp.%d" % os.getpid()
        _run([HIPCC] + LINK_FLAGS + ["-o", tmp] + objs, verbose)
        os.replace(tmp, LIB)
    finally:
        shutil.rmtree(work, ignore_errors=True)
    build_binding(verbose)
    return LIB


def build_binding(verbose=False):
    """Build the native part of the binding, which calls libscc_hip.so beside it."""
    import torch
    root = os.path.dirname(torch.__file__)
    includes = [os.path.join(root, "include"), os.path.join(root, "include", "torch", "csrc", "api", "include"),
                os.path.join(rocm_root(), "include"), sysconfig.get_paths()["include"], INCLUDE]
    tmp = BINDING_LIB + ".tmp.%d" % os.getpid()
    _run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
          "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI, '-DSCC_BUILT_FOR="%s"' % binding_tag()] + ["-I" + i for i in includes] +
         [BINDING_SRC, "-o", tmp, "-L" + os.path.join(root, "lib"), "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python",
          "-L" + HERE, "-lscc_hip", "-Wl,-rpath,$ORIGIN"], verbose)
    os.replace(tmp, BINDING_LIB)
    return BINDING_LIB


def build_membw(force=True, verbose=False):
    """Build libscc_membw.so, the plain copy / read kernels bench.py measures its copy ceiling with."""
    if not force and os.path.exists(MEMBW_LIB) and os.path.getmtime(MEMBW_LIB) >= os.path.getmtime(MEMBW_SRC):
        return MEMBW_LIB
    tmp = MEMBW_LIB + ".tmp.%d" % os.getpid()
    _run([HIPCC] + COMPILE_FLAGS + ["-shared", "-o", tmp, MEMBW_SRC], verbose)
    os.replace(tmp, MEMBW_LIB)
    return MEMBW_LIB


if __name__ == "__main__":
    print(build(force=True, verbose=True))
    print(build_membw(force=True, verbose=True))
