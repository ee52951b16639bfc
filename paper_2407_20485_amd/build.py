"""Builds liba2sf.so (HIP kernels + C ABI), _call.so (argument marshalling of binding.py, host code) and the
stand-alone `ceilings` probe (machine ceilings the roofline figures are compared with) for gfx950 next to this file.

    python -m paper_2407_20485_amd.build
"""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "liba2sf.so")
CALL = os.path.join(HERE, "_call.so")
CEILINGS = os.path.join(HERE, "ceilings")
SOURCES = ["a2sf_api.hip", "decode.hip", "select_compact.hip", "prefill_f32.hip", "prefill_bf16.hip",
           "similarity.hip", "chunk.hip"]
# -packed-fp32-ops is switched off: packed fp32 forms have produced wrong results on the
# target machines; the host pass does not know the feature and says so (harmless).
COMMON = ["--offload-arch=gfx950", "-O3", "-std=c++17",
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
          "-Wno-unused-command-line-argument"]
FLAGS = COMMON + ["-fPIC", "-shared"]


def generate() -> None:
    """Writes the generated instruction stream(s) the kernels include."""
    subprocess.run([sys.executable, os.path.join(CSRC, "gen_attn_fwd128x2.py")], check=True,
                   capture_output=True)


def _compile(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in res.stderr.splitlines() if noise not in l)
    if res.returncode != 0:
        raise RuntimeError(f"{cmd[0]} failed ({res.returncode}):\n{err}")
    if verbose and err.strip():
        print(err, file=sys.stderr)


def build_call(verbose: bool = False) -> str:
    """The host extension: g++ against torch's headers (torch's libraries are in the process when it is loaded)."""
    import torch

    home = os.path.dirname(torch.__file__)
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-w",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           "-I" + sysconfig.get_paths()["include"], "-I" + os.path.join(home, "include"),
           "-I" + os.path.join(home, "include", "torch", "csrc", "api", "include"), os.path.join(CSRC, "py_call.cpp"),
           "-L" + os.path.join(home, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-o", CALL]
    _compile(cmd, verbose)
    return CALL


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    generate()
    _compile([hipcc, *FLAGS, *[os.path.join(CSRC, s) for s in SOURCES], "-o", LIB], verbose)
    build_call(verbose)
    _compile([hipcc, *COMMON, os.path.join(CSRC, "ceilings.hip"), "-o", CEILINGS], verbose)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
