"""Build libmoss_hip.so (gfx950) in-tree with hipcc, and the native calls of the binding, _moss_calls.so, with the host
compiler.  `python -m paper_2511_05811_amd.build`."""
import hashlib
import os
import subprocess
import sys
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(os.path.dirname(PKG), "include")
LIB = os.path.join(PKG, "libmoss_hip.so")
CALLS = os.path.join(PKG, "_moss_calls.so")
SOURCES = ["moss_api.hip", "moss_quant.hip", "moss_weight.hip", "moss_gemm.hip", "moss_gemm_big.hip", "moss_gemm_mid.hip", "moss_swiglu.hip", "moss_rmsnorm.hip"]

FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
         "-ffp-contract=off",                      # numerically specified kernels: no FMA contraction
         "-fhip-fp32-correctly-rounded-divide-sqrt",  # IEEE '/' and sqrtf in device code
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument", "-Wno-inline-asm"]   # (the copies name M0 as clobbered: reserved, hence a warning)


def interface():
    """The number that the library and the native calls compiled against it share: of the headers that declare its functions."""
    h = hashlib.sha256()
    for path in (os.path.join(INCLUDE, "moss.h"), os.path.join(CSRC, "moss_producer.h")):
        with open(path, "rb") as f:
            h.update(f.read())
    return int(h.hexdigest()[:8], 16) | 1        # (never 0)


def build(verbose=False):
    """The library, and the native calls if they can be built: the binding works without them, so that hipcc is all it takes.  Native
    calls of an earlier build do not stay beside the new library."""
    if os.path.exists(CALLS):
        os.remove(CALLS)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc] + FLAGS + [f"-DMOSS_INTERFACE={interface()}u", "-I", INCLUDE, "-o", LIB] + [os.path.join(CSRC, s) for s in SOURCES]
    if verbose:
        print(" ".join(cmd))
    res = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in res.stderr.splitlines() if "is not a recognized feature" not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + err)
    if verbose and err.strip():
        print(err, file=sys.stderr)
    try:
        build_calls(verbose)
    except (OSError, ImportError, RuntimeError) as e:
        print(f"no native calls for the binding ({e}): it makes them from Python", file=sys.stderr)
    return LIB


def build_calls(verbose=False):
    """_moss_calls.so: needs torch's headers and links against the torch that is installed here."""
    import torch
    home = os.path.dirname(torch.__file__)
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}",
           f"-DMOSS_INTERFACE={interface()}u", f'-DMOSS_TORCH_VERSION="{torch.__version__}"',
           "-I", INCLUDE, "-I", CSRC, "-isystem", os.path.join(home, "include"), "-isystem", sysconfig.get_paths()["include"], "-o", CALLS,
           os.path.join(CSRC, "moss_calls.cpp"), "-L", os.path.join(home, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"]
    if verbose:
        print(" ".join(cmd))
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("building _moss_calls failed:\n" + res.stderr)


if __name__ == "__main__":
    print(build(verbose=True))
