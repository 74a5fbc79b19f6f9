"""Builds and calls dispatch_probe.cpp: which kernels the library's host layer
would launch for a call of the C ABI, with which plan (CPU only)."""
from __future__ import annotations

import ctypes
import functools
import os
import subprocess
import tempfile

import paper_2305_17190_amd as pam
from paper_2305_17190_amd import build

KERNELS = {1: "tiled", 2: "few rows", 3: "small", 4: "exact", 5: "reduce", 6: "fill"}


class Launch(ctypes.Structure):
    _fields_ = [(name, ctypes.c_int64) for name in ("kernel", "tile_m", "tile_n", "kgroups", "splits", "k_per_split",
                                                    "whole", "split_tiles", "few_rows_of_a", "batch")]

    @property
    def name(self) -> str:
        return KERNELS[self.kernel]


@functools.lru_cache(maxsize=None)
def library() -> ctypes.CDLL:
    here = os.path.dirname(os.path.abspath(__file__))
    with tempfile.TemporaryDirectory() as tmp:
        so = os.path.join(tmp, "dispatch_probe.so")
        rocm = os.path.join(os.path.dirname(os.path.dirname(build.hipcc())), "include")
        subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-fPIC", "-shared", "-Wl,-Bsymbolic", "-D__HIP_PLATFORM_AMD__",
                        "-isystem", rocm, "-I", build.INCLUDE, "-I", build.CSRC,
                        os.path.join(here, "dispatch_probe.cpp"), "-o", so], check=True)
        lib = ctypes.CDLL(so)
    real = pam.load()
    for name in pam.EXPORTS:
        getattr(lib, name).argtypes = getattr(real, name).argtypes
        getattr(lib, name).restype = getattr(real, name).restype
    lib.probe_take.argtypes = [ctypes.POINTER(Launch)]
    lib.probe_take.restype = ctypes.c_int
    return lib


def _launches():
    out = (Launch * 8)()
    return list(out[:library().probe_take(out)])


PTR = 1 << 20   # stands for every device address


def product(m, n, k, batch=1, ta=False, tb=True, workspace=True, plan=None, bf16=False):
    """The launches of a product with dense operands: the library's choice with
    a workspace or without one, or under `plan`."""
    lib = library()
    lda, ldb = max(1, m if ta else k), max(1, k if tb else n)
    args = (int(ta), int(tb), m, n, k, PTR, lda, m * k, PTR, ldb, k * n, PTR, n, m * n, batch)
    if plan is not None:
        p = pam._Plan(*plan)
        status = lib.pam_gemm_batched_with_plan(*args, ctypes.byref(p), PTR, 1 << 60, None)
    elif bf16:
        status = lib.pam_gemm_batched_bf16(*args, PTR if workspace else None, 1 << 60, None)
    elif workspace:
        status = lib.pam_gemm_batched_ws(*args, 23, PTR, 1 << 60, None)
    else:
        status = lib.pam_gemm_batched(*args, None)
    assert status == 0, lib.pam_last_error()
    return _launches()


def exact_grad(m, n, k, workspace=True):
    """The launches of an exact-derivative product."""
    lib = library()
    args = (0, m, n, k, PTR, max(1, k), PTR, n, PTR, n, PTR, n)
    if workspace:
        status = lib.pam_gemm_exact_grad_ws(*args, PTR, 1 << 60, None)
    else:
        status = lib.pam_gemm_exact_grad(*args, None)
    assert status == 0, lib.pam_last_error()
    return _launches()


def plan(m, n, k, batch=1, max_workspace_bytes=None):
    """As paper_2305_17190_amd.plan, from the probe's host layer."""
    p = pam._Plan()
    limit = (1 << 64) - 1 if max_workspace_bytes is None else max_workspace_bytes
    assert library().pam_gemm_plan_for_workspace(m, n, k, batch, limit, ctypes.byref(p)) == 0
    return (p.tile_m, p.tile_n, p.splits, p.kgroups, p.whole_tiles)
