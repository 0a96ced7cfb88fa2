"""Build the HIP library in-tree for gfx950: `python -m paper_2603_02170_amd.build`."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "libsagebwd.so")
HOST = os.path.join(HERE, "_sage_host.so")


def hipcc_path() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.sep not in cand or os.path.exists(cand)):
            return cand
    return "hipcc"


def _run(cmd, verbose: bool) -> None:
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    out = "\n".join(l for l in (res.stdout + res.stderr).splitlines()
                    if "packed-fp32-ops" not in l and "is not a recognized feature" not in l)
    if res.returncode != 0:
        raise RuntimeError(f"{os.path.basename(cmd[0])} failed:\n" + out)
    if verbose and out.strip():
        print(out)


def build(verbose: bool = True) -> str:
    """Compile csrc/sagebwd_api.hip (which includes every kernel) into libsagebwd.so, and csrc/torch_host.cpp
    (host code only: what stands between Python's tensors and that library) into _sage_host.so."""
    src = os.path.join(HERE, "csrc", "sagebwd_api.hip")
    cmd = [
        hipcc_path(), "--offload-arch=gfx950", "-O3", "-std=c++17", "-shared", "-fPIC",
        # packed FP32 instructions are kept out of the generated code on purpose
        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
        "-Wno-unused-command-line-argument",
        "-I", os.path.join(ROOT, "include"), "-I", os.path.join(HERE, "csrc"),
        src, "-o", LIB,
    ]
    cmd[1:1] = os.environ.get("SAGEBWD_EXTRA_CFLAGS", "").split()   # e.g. -DNAME for kernel experiments
    _run(cmd, verbose)
    build_host(verbose)
    return LIB


def build_host(verbose: bool = True) -> str:
    import sysconfig

    import torch
    from torch.utils import cpp_extension
    torch_lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-shared", "-fPIC", "-fvisibility=hidden",
           "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}"]
    for inc in cpp_extension.include_paths() + [sysconfig.get_paths()["include"], "/opt/rocm/include"]:
        cmd += ["-isystem", inc]
    cmd += ["-I", os.path.join(ROOT, "include"), os.path.join(HERE, "csrc", "torch_host.cpp"), "-o", HOST,
            "-L", HERE, "-l:libsagebwd.so", "-Wl,-rpath,$ORIGIN",
            "-L", torch_lib, "-ltorch_python", "-ltorch_cpu", "-ltorch_hip", "-ltorch", "-lc10_hip", "-lc10"]
    _run(cmd, verbose)
    return HOST


if __name__ == "__main__":
    build()
    print("built", LIB)
    sys.exit(0)
