"""Compile the HIP sources into paper_1710_03740_amd/libmpt.so for gfx950, and the binding's native calls into _calls.so.

Run as `python -m paper_1710_03740_amd.build`.  hipcc cross-compiles without a
GPU.  Both are built in-tree so that they travel with the source tree.
"""
import os
import shutil
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
LIB = os.path.join(HERE, "libmpt.so")
CALLS = os.path.join(HERE, "_calls.so")
OBJDIR = os.path.join(HERE, "_build")

HIP_SOURCES = ["elementwise.hip", "gemm.hip", "gemm_ring.hip", "norm.hip", "optim.hip", "lstm.hip", "probe.hip"]
CXX_SOURCES = ["host.cpp"]

# -ffp-contract=off: the update path is specified as separately rounded FP32 operations.
# packed-fp32 VALU forms are disabled for the whole library.
HIP_FLAGS = ["-O3", "--offload-arch=gfx950", "-fPIC", "-std=c++17", "-ffp-contract=off",
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
             "-Wno-unused-command-line-argument", "-I", INCLUDE, "-I", CSRC]


def _calls_missing():
    """What it takes to compile the native calls and is not here, or None.  The library itself needs hipcc only."""
    if shutil.which("g++") is None:
        return "g++"
    try:
        from torch.utils import cpp_extension
    except ImportError:
        return "torch"
    for header in ("torch/csrc/autograd/python_variable.h", "Python.h"):
        if not any(os.path.exists(os.path.join(d, header)) for d in (*cpp_extension.include_paths(), sysconfig.get_path("include"))):
            return header
    return None


def _calls_command():
    """The extension module that unpacks torch's tensors: host code against the installed torch's headers."""
    import torch
    from torch.utils import cpp_extension
    from . import binding
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    inc = [*cpp_extension.include_paths(), os.path.join(rocm, "include"), sysconfig.get_path("include")]
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    return (["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wextra", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
             "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI, '-DMPT_TORCH="%s"' % binding.torch_build(), "-I" + INCLUDE]
            + ["-isystem" + d for d in inc] + [os.path.join(CSRC, "calls.cpp"), "-o", CALLS, "-L" + lib, "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"])


def _run(cmd):
    p = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in p.stdout.splitlines() if "packed-fp32-ops" not in l)
    if p.returncode != 0:
        raise RuntimeError("build failed: %s\n%s" % (" ".join(cmd), out))
    if out.strip():
        print(out)


def build(verbose=True):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(OBJDIR, exist_ok=True)
    objs = []
    procs = []
    for src in HIP_SOURCES + CXX_SOURCES:
        path = os.path.join(CSRC, src)
        if not os.path.exists(path):
            raise RuntimeError("missing source " + path)
        obj = os.path.join(OBJDIR, src + ".o")
        objs.append(obj)
        lang = ["-x", "hip"] if src.endswith(".hip") else []
        cmd = [hipcc] + HIP_FLAGS + lang + ["-c", path, "-o", obj]
        if verbose:
            print("[mpt build]", src, flush=True)
        procs.append((cmd, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    missing = _calls_missing()
    if missing is None:
        cmd = _calls_command()
        if verbose:
            print("[mpt build] calls.cpp", flush=True)
        procs.append((cmd, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    else:
        print("[mpt build] no %s here: without %s, calls go through ctypes" % (missing, os.path.basename(CALLS)), flush=True)
        if os.path.exists(CALLS):
            os.remove(CALLS)                      # it may know another library's entry points
    for cmd, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode != 0:
            raise RuntimeError("build failed: %s\n%s" % (" ".join(cmd), out))
        if out.strip() and verbose:
            print(out)
    _run([hipcc, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", LIB] + objs)
    if verbose:
        print("[mpt build] wrote", LIB, *([CALLS] if missing is None else []), flush=True)
    return LIB


if __name__ == "__main__":
    build()
    sys.exit(0)
