"""Build libkroquant.so in-tree with hipcc for gfx950 (no JIT cache)."""
from __future__ import annotations

import os
import subprocess
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libkroquant.so")
BIND = os.path.join(PKG, "_kqbind.so")  # native marshalling of the Python binding
SOURCES = ["kq_kernels.hip", "kq_gemm.hip", "kq_calib.hip", "kq_api.hip"]

# -packed-fp32-ops off: no v_pk_{add,mul,fma}_f32 in the device code.
# -ffp-contract=off: only the explicit fmaf calls fuse, which keeps the
# evaluation order of the arithmetic contract in kq_kernels.hip.
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-ffp-contract=off",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # matrix-core results in architectural VGPRs (no accumulator-register reads)
    "-mllvm", "-amdgpu-mfma-vgpr-form=true",
    "-Wall", "-Wno-unused-command-line-argument",
]


def hipcc() -> str:
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    return os.path.join(rocm, "bin", "hipcc")


def _run(cmd: list[str], verbose: bool) -> None:
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"{cmd[0]} failed ({res.returncode}):\n{res.stdout}\n{res.stderr}")


def build_bind(verbose: bool = False) -> str:
    """Compile the Python binding's native part against torch and libkroquant.so."""
    import torch
    from torch.utils.cpp_extension import include_paths
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    inc = [*include_paths(), os.path.join(rocm, "include"), sysconfig.get_paths()["include"], os.path.join(ROOT, "include")]
    _run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", "-w",
          *[a for i in inc for a in ("-isystem", i)], os.path.join(CSRC, "kq_bind.cpp"),
          "-L" + PKG, "-l:libkroquant.so", "-Wl,-rpath,$ORIGIN",
          "-L" + os.path.join(os.path.dirname(torch.__file__), "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip", "-o", BIND + ".tmp"], verbose)
    os.replace(BIND + ".tmp", BIND)
    return BIND


def build(verbose: bool = False) -> str:
    """Compile every HIP source into libkroquant.so (always recompiles), then the binding's native part."""
    cmd = [hipcc(), *HIPCC_FLAGS, "-I", os.path.join(ROOT, "include"), "-I", CSRC,
           *[os.path.join(CSRC, s) for s in SOURCES], "-o", LIB + ".tmp"]
    _run(cmd, verbose)
    os.replace(LIB + ".tmp", LIB)
    build_bind(verbose)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
