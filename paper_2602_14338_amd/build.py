"""Builds the gfx950 shared library in-tree with hipcc, and the binding's native marshalling module (host code)
against torch's headers.  No JIT cache."""
import os
import subprocess
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libaero_hip.so")
MARSHAL = os.path.join(PKG, "_marshal.so")
SOURCES = ["aero_api.hip", "group_advantage.hip", "logprob_fwd.hip", "grpo_loss_bwd.hip", "grpo_single_pass.hip",
           "lmhead_fused.hip"]
FLAGS = ["-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC", "-shared",
         # keep the compiler from forming packed-fp32 VALU ops from scalar float code
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function"]


def _run(cmd, verbose: bool) -> None:
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in r.stdout.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(os.path.basename(cmd[0]) + " failed:\n" + out)
    if verbose and out.strip():
        print(out)


def build_marshal(verbose: bool = False) -> str:
    import torch
    from torch.utils import cpp_extension
    inc = cpp_extension.include_paths() + [sysconfig.get_paths()["include"]]
    lib_dir = os.path.join(os.path.dirname(torch.__file__), "lib")
    _run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared",
          f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}"] + [f"-I{i}" for i in inc] +
         [os.path.join(CSRC, "marshal.cpp"), "-o", MARSHAL, "-L" + lib_dir, "-ltorch_python", "-ltorch_cpu", "-lc10"],
         verbose)
    return MARSHAL


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    _run([hipcc] + FLAGS + [os.path.join(CSRC, s) for s in SOURCES] + ["-o", LIB], verbose)
    build_marshal(verbose)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
