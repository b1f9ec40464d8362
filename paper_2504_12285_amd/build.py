"""Builds libbitlinear_hip.so (HIP kernels + C-ABI, gfx950) in-tree with hipcc, and _bl_torch.so (the binding's small
calls, host code against the installed torch) with g++."""
import os
import subprocess
import sysconfig

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG_DIR, "csrc")
INCLUDE = os.path.join(os.path.dirname(PKG_DIR), "include")
LIB_PATH = os.path.join(PKG_DIR, "libbitlinear_hip.so")
TORCH_EXT_PATH = os.path.join(PKG_DIR, "_bl_torch.so")
TORCH_EXT_SOURCE = os.path.join(CSRC, "bl_torch.cpp")
SOURCES = ["bl_api.cpp", "bl_pack.hip", "bl_quant.hip", "bl_gemv.hip", "bl_gemv_one.hip", "bl_gemv_panel.hip", "bl_gemm.hip", "bl_stream.hip", "bl_probe.hip"]
HIPCC_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-ffp-contract=off",
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def sources():
    return [os.path.join(CSRC, s) for s in SOURCES]


def is_stale():
    if not os.path.exists(LIB_PATH) or not os.path.exists(TORCH_EXT_PATH):
        return True
    if os.path.getmtime(TORCH_EXT_SOURCE) > os.path.getmtime(TORCH_EXT_PATH):
        return True
    t = os.path.getmtime(LIB_PATH)
    deps = sources() + [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".h")]
    deps.append(os.path.join(INCLUDE, "bitlinear.h"))
    return any(os.path.getmtime(d) > t for d in deps)


def build_torch_ext(verbose=False):
    """Compile the native form of the binding's small calls."""
    import torch
    root = os.path.dirname(torch.__file__)
    tmp = TORCH_EXT_PATH + ".tmp%d" % os.getpid()
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI]
    for d in (INCLUDE, os.path.join(root, "include"), os.path.join(root, "include", "torch", "csrc", "api", "include"),
              sysconfig.get_paths()["include"], os.path.join(rocm, "include")):
        cmd += ["-I", d]
    cmd += ["-o", tmp, TORCH_EXT_SOURCE, "-L", os.path.join(root, "lib"), "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"]
    if verbose:
        print(" ".join(cmd))
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if res.returncode != 0:
        raise RuntimeError("g++ failed:\n" + res.stdout)
    os.replace(tmp, TORCH_EXT_PATH)
    return TORCH_EXT_PATH


def build(verbose=False):
    """Compile every HIP source for gfx950 into one shared library, and the torch side of the binding."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = LIB_PATH + ".tmp%d" % os.getpid()
    cmd = [hipcc] + HIPCC_FLAGS + ["-I", INCLUDE, "-I", CSRC, "-o", tmp] + sources()
    if verbose:
        print(" ".join(cmd))
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # the host pass does not know the packed-fp32 feature switch; that note is harmless
    out = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + out)
    if verbose and out.strip():
        print(out)
    os.replace(tmp, LIB_PATH)
    build_torch_ext(verbose)
    return LIB_PATH


if __name__ == "__main__":
    build(verbose=True)
