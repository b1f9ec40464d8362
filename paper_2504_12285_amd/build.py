"""Builds libbitlinear_hip.so (HIP kernels + C-ABI, gfx950) in-tree with hipcc, and the _bl_torch extension (the binding's
small calls, host code against the installed torch) with g++."""
import importlib.metadata
import os
import shutil
import subprocess
import sysconfig
import warnings

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG_DIR, "csrc")
INCLUDE = os.path.join(os.path.dirname(PKG_DIR), "include")
LIB_PATH = os.path.join(PKG_DIR, "libbitlinear_hip.so")
TORCH_EXT_PATH = os.path.join(PKG_DIR, "_bl_torch" + sysconfig.get_config_var("EXT_SUFFIX"))   # of this interpreter
TORCH_EXT_SOURCE = os.path.join(CSRC, "bl_torch.cpp")
SOURCES = ["bl_api.cpp", "bl_pack.hip", "bl_quant.hip", "bl_gemv.hip", "bl_gemv_one.hip", "bl_gemv_panel.hip", "bl_gemm.hip", "bl_stream.hip", "bl_probe.hip"]
HIPCC_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-ffp-contract=off",
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
               # The first 14 scalar registers of a kernel's arguments are in place when its waves start.  bl_gemv_one is laid out for
               # it; over sweeps of the entry points the time with it against without: one token x one matrix 0.99 - 1.00, quantisers 0.97 - 1.00
               # (one row 1.00 - 1.03), prefill tiles 0.99, fused epilogues and the split k loop 1.01, decode of 2 to 64 tokens
               # 1.00 - 1.01, packing 1.00 - 1.02 (those two vary as much between builds of the same code).
               "-mllvm", "-amdgpu-kernarg-preload-count=14"]


def sources():
    return [os.path.join(CSRC, s) for s in SOURCES]


def torch_version():
    """The installed torch, without importing it; None without one."""
    try:
        return importlib.metadata.version("torch")
    except importlib.metadata.PackageNotFoundError:
        return None


def _torch_mark():
    """What the extension carries of the torch that it was built against (BL_TORCH_VERSION in bl_torch.cpp)."""
    return b"built for torch " + str(torch_version()).encode() + b"\0"


def torch_ext_missing():
    """Why the extension cannot be built here, or None.  The library does without it."""
    if shutil.which("g++") is None:
        return "no g++"
    if torch_version() is None:
        return "no torch"
    if not os.path.exists(os.path.join(sysconfig.get_paths()["include"], "Python.h")):
        return "no Python.h"
    return None


def _older(path, deps):
    return not os.path.exists(path) or any(os.path.getmtime(d) > os.path.getmtime(path) for d in deps)


def _headers():
    """The headers, and this file, which holds the flags."""
    return [os.path.abspath(__file__), os.path.join(INCLUDE, "bitlinear.h")] + [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".h")]


def torch_ext_is_stale():
    if _older(TORCH_EXT_PATH, [TORCH_EXT_SOURCE, os.path.join(INCLUDE, "bitlinear.h"), os.path.abspath(__file__)]):
        return True
    with open(TORCH_EXT_PATH, "rb") as f:
        return _torch_mark() not in f.read()


def is_stale():
    return _older(LIB_PATH, sources() + _headers()) or (torch_ext_missing() is None and torch_ext_is_stale())


def _compile(cmd, what, verbose):
    if verbose:
        print(" ".join(cmd))
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # the host pass does not know the packed-fp32 feature switch; that note is harmless
    out = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError(what + " failed:\n" + out)
    if verbose and out.strip():
        print(out)


def _torch_ext_command(out):
    import torch
    root = os.path.dirname(torch.__file__)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI, '-DBL_TORCH_VERSION="%s"' % torch_version()]
    for d in (INCLUDE, os.path.join(root, "include"), os.path.join(root, "include", "torch", "csrc", "api", "include"),
              sysconfig.get_paths()["include"], os.path.join(rocm, "include")):
        cmd += ["-I", d]
    return cmd + ["-o", out, TORCH_EXT_SOURCE, "-L", os.path.join(root, "lib"), "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"]


def _install(new, ext):
    """Puts the compiled files in place, an extension never beside a library that it was not built with."""
    for f in os.listdir(PKG_DIR):
        if f.startswith("_bl_torch.") and f.endswith(".so"):
            os.remove(os.path.join(PKG_DIR, f))
    os.replace(new, LIB_PATH)
    if ext:
        os.replace(ext, TORCH_EXT_PATH)


def build(verbose=False):
    """Compile every HIP source for gfx950 into one shared library, and the torch side of the binding where its
    tools are there (the binding does without it, more slowly)."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp, ext = LIB_PATH + ".tmp%d" % os.getpid(), TORCH_EXT_PATH + ".tmp%d" % os.getpid()
    why = torch_ext_missing()
    if why is None:
        _compile(_torch_ext_command(ext), "g++", verbose)
    else:
        warnings.warn("the binding's native form is not built: " + why, RuntimeWarning)
    _compile([hipcc] + HIPCC_FLAGS + ["-I", INCLUDE, "-I", CSRC, "-o", tmp] + sources(), "hipcc", verbose)
    _install(tmp, ext if why is None else None)
    return LIB_PATH


if __name__ == "__main__":
    build(verbose=True)
