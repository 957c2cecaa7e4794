"""Builds libmqa_decode.so (gfx950) with hipcc and the binding's native calls in-tree.  `python -m paper_1911_02150_amd.build`."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG_DIR, "csrc")
LIB_PATH = os.path.join(PKG_DIR, "libmqa_decode.so")
SOURCES = ["api.hip", "decode_mfma.hip", "decode_direct.hip", "prompt_mfma.hip", "decode_generic.hip", "small_kernels.hip", "project.hip", "project_kv.hip", "project_kv_rows.hip", "project_terms.hip", "gemm.hip", "packed.hip", "stack_kernels.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument", "-Wno-unknown-attributes",
]


CALLS_PATH = os.path.join(PKG_DIR, "_calls" + sysconfig.get_config_var("EXT_SUFFIX"))      # (another Python does not load it)


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    out = "\n".join(l for l in (res.stdout + res.stderr).splitlines()
                    if "packed-fp32-ops" not in l)          # host pass does not know the GPU feature
    if verbose and out.strip():
        print(out, flush=True)
    if res.returncode != 0:
        raise RuntimeError(f"{os.path.basename(cmd[0])} failed:\n" + out)


def build_calls(verbose: bool = True) -> str:
    """The binding's native calls: host code over torch's tensor type."""
    import torch
    torch_dir = os.path.dirname(torch.__file__)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    includes = [os.path.join(torch_dir, "include"), os.path.join(torch_dir, "include", "torch", "csrc", "api", "include"),
                sysconfig.get_paths()["include"], os.path.join(rocm, "include")]
    _run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-shared", "-fPIC", "-Wall", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
          "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", f'-DMQA_TORCH_VERSION="{torch.__version__}"', *[f"-I{d}" for d in includes], os.path.join(CSRC, "calls.cpp"), "-o", CALLS_PATH,
          f"-L{os.path.join(torch_dir, 'lib')}", "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"], verbose)
    return CALLS_PATH


def build_library(verbose: bool = True, extra_flags=()) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *HIPCC_FLAGS, *extra_flags, *[os.path.join(CSRC, s) for s in SOURCES], "-o", LIB_PATH]
    _run(cmd, verbose)
    return LIB_PATH


if __name__ == "__main__":
    build_library()
    build_calls()
    sys.exit(0)
