"""Build libtiled_sdpa.so (gfx950 only) from csrc/*.hip with hipcc, objects in parallel, and _torch_calls.so (the
tensor entry points, host code only) from csrc/torch_calls.cpp with g++ against torch's headers.

Usage: python -m paper_2603_01960_amd.build [--force]
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor
from pathlib import Path

PKG = Path(__file__).resolve().parent
CSRC = PKG / "csrc"
INCLUDE = PKG.parent / "include"
OBJ = PKG / "_build"
LIB = PKG / "libtiled_sdpa.so"
CALLS_SRC = CSRC / "torch_calls.cpp"
CALLS = PKG / "_torch_calls.so"

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
    # packed FP32 VALU forms are kept out of the generated code on purpose
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unknown-warning-option",
    f"-I{INCLUDE}", f"-I{CSRC}",
]

# The forward kernels on 64-row K/V tiles (up to D = 128) are scheduled by LLVM's iterative ILP
# strategy: measured 3-5 % faster than the default on every one of them.  The same strategy halves the
# speed of the 32-row tile kernels (it lengthens live ranges past their 168-register budget).  The backward
# kernels gain 1-5 % from it at D = 64, 96 and 160; at D = 128, where the fused dK + dV pass has two registers
# left, it spills and loses 2-10 %.  So it is applied per translation unit and never elsewhere.
ILP_SCHED = ["-mllvm", "-amdgpu-sched-strategy=iterative-ilp"]


# The five-product backward keeps dK and dV in accumulation registers by itself and everything else out of them:
# left to its own choice, the compiler puts the results of all matrix instructions there once one is, and copies.
MFMA_VGPR = ["-mllvm", "-amdgpu-mfma-vgpr-form=1"]


def extra_flags(src: Path) -> list[str]:
    name = src.name
    if name.startswith("sdpa_bwd_chain_"):
        return MFMA_VGPR
    if name.startswith("sdpa_fwd_") and name.endswith("_tn64.hip") and "_d160_" not in name:
        return ILP_SCHED
    if name.startswith("sdpa_bwd_") and not name.endswith("_d128.hip"):
        return ILP_SCHED
    return []


def sources():
    return sorted(CSRC.glob("*.hip"))


def _compile(src: Path) -> Path:
    obj = OBJ / (src.stem + ".o")
    cmd = [HIPCC, *FLAGS, *extra_flags(src), "-c", str(src), "-o", str(obj)]
    res = subprocess.run(cmd, capture_output=True, text=True)
    noise = ("packed-fp32-ops", "is not a recognized feature")
    err = "\n".join(l for l in res.stderr.splitlines() if not any(n in l for n in noise))
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src.name}:\n{err}")
    if err.strip():
        print(err, file=sys.stderr)
    return obj


def build_calls() -> Path:
    """The CPython module behind the tensor functions of binding.py; links against LIB, which must exist."""
    import sysconfig

    import torch

    root = Path(torch.__file__).resolve().parent
    rocm = Path(HIPCC).resolve().parents[1]
    tmp = CALLS.with_suffix(f".tmp{os.getpid()}.so")
    # (the two definitions are what ROCm's and torch's headers expect of a host compiler other than hipcc)
    subprocess.run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-w",
                    "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
                    f"-I{INCLUDE}", f"-I{root / 'include'}", f"-I{root / 'include/torch/csrc/api/include'}",
                    f"-I{rocm / 'include'}", f"-I{sysconfig.get_paths()['include']}",
                    str(CALLS_SRC), "-o", str(tmp), f"-L{PKG}", f"-L{root / 'lib'}",
                    "-ltiled_sdpa", "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_hip", "-ltorch_python",
                    "-Wl,-rpath,$ORIGIN"], check=True)
    os.replace(tmp, CALLS)
    return CALLS


def build(force: bool = True, jobs: int | None = None) -> Path:
    OBJ.mkdir(exist_ok=True)
    srcs = sources()
    headers = list(CSRC.glob("*.h")) + list(INCLUDE.glob("*.h"))
    newest = max(p.stat().st_mtime for p in [*srcs, *headers, CALLS_SRC])
    if not force and all(p.exists() and p.stat().st_mtime >= newest for p in (LIB, CALLS)):
        return LIB
    jobs = jobs or min(len(srcs), int(os.environ.get("MAX_JOBS", os.cpu_count() or 4)), 16)
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(_compile, srcs))
    tmp = LIB.with_suffix(f".tmp{os.getpid()}.so")
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-fno-gpu-rdc",
                    *map(str, objs), "-o", str(tmp)], check=True)
    os.replace(tmp, LIB)
    build_calls()
    return LIB


if __name__ == "__main__":
    print(build(force="--force" in sys.argv or True))
