"""Build step for the HIP library libpam.so (gfx950 only).

    python -m paper_2305_17190_amd.build

compiles csrc/*.hip and csrc/*.cpp with hipcc into paper_2305_17190_amd/libpam.so,
one object per source (the matrix product kernels in PARTS of their source),
several at a time.
"""
from __future__ import annotations

import concurrent.futures
import os
import shutil
import subprocess
import sys
import tempfile

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(PKG, "libpam.so")

# Device code: gfx950 only; float32 denormals flushed (the GEMM relies on the
# accumulate treating denormal encodings as zero); no packed-fp32 VALU ops.
DEVICE_FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fgpu-flush-denormals-to-zero",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def hipcc() -> str:
    path = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(path):
        raise RuntimeError("hipcc not found; the PAM library needs ROCm's hipcc")
    return path


def sources():
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith((".hip", ".cpp")))


# Sources compiled in parts, one object each (their count of parts).
PARTS = {"pam_gemm_dma.hip": 6}


def _run(cmd, verbose: bool) -> None:
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + res.stderr)
        raise RuntimeError("hipcc failed to build libpam.so")


def build(verbose: bool = False, extra_flags=()) -> str:
    flags = [hipcc(), *DEVICE_FLAGS, *extra_flags, "-fPIC"]
    with tempfile.TemporaryDirectory() as tmpdir:
        jobs = []
        for src in sources():
            name = os.path.basename(src)
            for part in range(PARTS.get(name, 1)):
                obj = os.path.join(tmpdir, f"{name}.{part}.o")
                define = [f"-DPAM_GEMM_PART={part}"] if name in PARTS else []
                jobs.append(([*flags, *define, "-I", INCLUDE, "-I", CSRC, "-c", src, "-o", obj], obj))
        with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as pool:
            for done in [pool.submit(_run, cmd, verbose) for cmd, _ in jobs]:
                done.result()
        tmp = f"{LIB}.{os.getpid()}.tmp"   # per process: concurrent builds never see a partial file
        _run([*flags, "-shared", *(obj for _, obj in jobs), "-o", tmp, "-lhsa-runtime64"], verbose)
        os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
