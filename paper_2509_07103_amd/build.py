"""Build the HIP library (liblmkan.so) for gfx950, and the extension module that marshals the calls to
it (_native.so), in-tree, next to this file."""
from __future__ import annotations

import glob
import os
import re
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "liblmkan.so")
NATIVE_SOURCE = os.path.join(CSRC, "lmkan_torch.cpp")
NATIVE = os.path.join(HERE, "_native.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# Packed float32 VALU instructions are switched off: some of their forms have given
# silently wrong results on the target machines.  MFMA accumulators are kept in ordinary
# vector registers (gfx950 allows it): the coefficient-gradient kernel reads them with
# vector instructions at the end of every cell, and copies out of the accumulation
# registers would cost as much as the combine itself.
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-mllvm", "-amdgpu-mfma-vgpr-form",
    "-munsafe-fp-atomics", "-Wall", "-Wno-unused-command-line-argument",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def sources() -> list[str]:
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def build(verbose: bool = False, extra: list[str] | None = None) -> str:
    """Compiles the library; the compiler's resource report of the same run goes through
    check_codegen.check_resources, so a build whose hot kernels spill registers raises."""
    cmd = [HIPCC, *FLAGS, "-Rpass-analysis=kernel-resource-usage", *(extra or []), "-o", LIB, *sources()]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + res.stderr)
        raise RuntimeError("hipcc failed building liblmkan.so")
    # (what is left of stderr without the report and the source lines it quotes: warnings)
    other = "\n".join(line for line in res.stderr.split("\n")
                      if "kernel-resource-usage" not in line and not re.match(r"\s*\d*\s*\|", line))
    if verbose and other.strip():
        sys.stderr.write(other)
    from . import check_codegen
    scratch = check_codegen.check_resources(res.stderr)
    if verbose:
        print(f"resource check: {len(scratch)} kernels, {sum(1 for v in scratch.values() if v)} with scratch "
              f"(at most {max(scratch.values())} bytes per lane)", flush=True)
    return LIB


def build_native() -> str:
    """Compiles the extension module (host code only) against the headers of the torch in use."""
    import torch
    base = os.path.dirname(torch.__file__)
    cmd = ["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-Wall", "-DUSE_ROCM", "-D__HIP_PLATFORM_AMD__=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           "-I", os.path.join(base, "include"), "-I", os.path.join(base, "include", "torch", "csrc", "api", "include"),
           "-I", "/opt/rocm/include", "-I", sysconfig.get_paths()["include"], "-I", os.path.join(ROOT, "include"),
           "-o", NATIVE, NATIVE_SOURCE,
           "-L", os.path.join(base, "lib"), "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + res.stderr)
        raise RuntimeError("g++ failed building _native.so")
    return NATIVE


def up_to_date() -> bool:
    if not os.path.exists(LIB) or not os.path.exists(NATIVE):
        return False
    t = min(os.path.getmtime(LIB), os.path.getmtime(NATIVE))
    deps = sources() + [NATIVE_SOURCE] + glob.glob(os.path.join(CSRC, "*.h")) + [os.path.join(ROOT, "include", "lmkan.h")]
    return all(os.path.getmtime(d) <= t for d in deps)


if __name__ == "__main__":
    print(build_native())
    print(build(verbose=True))
    sys.path.insert(0, ROOT)
    from paper_2509_07103_amd import check_codegen
    check_codegen.check(verbose=True)
    check_codegen.check(verbose=True, sources=check_codegen.SPARSE_SOURCES)
