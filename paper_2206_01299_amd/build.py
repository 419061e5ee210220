"""Build step: compile csrc/*.hip for gfx950 into ``libaqsgd.so`` beside this file, and
csrc/binding_native.cpp (host code, against torch's headers) into ``_native.so``.

Run as ``python -m paper_2206_01299_amd.build``.  hipcc cross-compiles without a
GPU.  Flags that matter for correctness:
  -ffp-contract=off   one rounding per written operation (the wire format)
  -packed-fp32-ops off  no packed binary32 instructions
and for launches:
  -amdgpu-kernarg-preload-count=14  a kernel's leading plain arguments arrive in scalar registers
"""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor
from pathlib import Path

HERE = Path(__file__).resolve().parent
CSRC = HERE / "csrc"
INCLUDE = HERE.parent / "include"
OBJDIR = HERE / "_build"
LIB = HERE / "libaqsgd.so"
NATIVE = HERE / "_native.so"

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-ffp-contract=off", "-fno-fast-math", "-fhip-fp32-correctly-rounded-divide-sqrt",
    "-fno-gpu-flush-denormals-to-zero",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-mllvm", "-amdgpu-kernarg-preload-count=14",
    "-Wall", "-Wno-unused-function", "-Wno-unknown-warning-option",
    f"-I{INCLUDE}", f"-I{CSRC}",
]


def sources():
    return sorted(CSRC.glob("*.hip"))


def _compile(src: Path) -> Path:
    obj = OBJDIR / (src.stem + ".o")
    cmd = [HIPCC, *FLAGS, "-c", str(src), "-o", str(obj)]
    res = subprocess.run(cmd, capture_output=True, text=True)
    noise = "packed-fp32-ops' is not a recognized feature"
    err = "\n".join(l for l in res.stderr.splitlines() if noise not in l)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src.name}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def _build_native() -> None:
    import torch
    t = Path(torch.__file__).resolve().parent
    tmp = NATIVE.with_suffix(f".tmp{os.getpid()}.so")
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-w",
           "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM", f"-I{sysconfig.get_paths()['include']}", f"-I{t}/include",
           f"-I{t}/include/torch/csrc/api/include", "-I/opt/rocm/include", f"-I{INCLUDE}",
           str(CSRC / "binding_native.cpp"), "-o", str(tmp),
           f"-L{t}/lib", "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]   # loaded by `import torch`
    if subprocess.run(cmd).returncode != 0:
        NATIVE.unlink(missing_ok=True)                  # none rather than an older one: calls take the ctypes path
        raise RuntimeError(f"the host compiler failed on binding_native.cpp ({LIB.name} works without it)")
    os.replace(tmp, NATIVE)


def build(verbose: bool = True) -> Path:
    OBJDIR.mkdir(exist_ok=True)
    srcs = sources()
    jobs = min(len(srcs), int(os.environ.get("MAX_JOBS", "8")), 16)
    with ThreadPoolExecutor(max_workers=jobs) as pool:
        native = pool.submit(_build_native)
        objs = list(pool.map(_compile, srcs))
    tmp = LIB.with_suffix(f".tmp{os.getpid()}.so")
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *map(str, objs), "-o", str(tmp)],
                   check=True)
    os.replace(tmp, LIB)
    native.result()                                     # a failure there leaves the library in place
    if verbose:
        print(f"built {LIB} from {len(srcs)} sources, and {NATIVE.name}")
    return LIB


if __name__ == "__main__":
    build()
