"""Build libkdtree.so (HIP for gfx950) in-tree with hipcc.

    python -m paper_2210_12859_amd.build

Every source is compiled to an object in ``_build/`` in parallel, then linked
into ``paper_2210_12859_amd/libkdtree.so``.  Floating-point flags keep the
squared distances bit-identical to plain IEEE binary32 arithmetic: no
contraction into FMA, denormals preserved; packed FP32 instructions are
disabled.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import re
import shutil
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
BUILD = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "libkdtree.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# (source, compiled for the device, extra flags)
SOURCES = [
    ("kd_api.cpp", True, []),
    ("kd_build_host.cpp", False, []),
    ("kd_traverse.hip", True, []),
    ("kd_packet.hip", True, ["-mllvm", "-amdgpu-mfma-vgpr-form"]),
    ("kd_wave.hip", True, []),
    ("kd_sort.hip", True, []),
    # matrix-core results in ordinary VGPRs (the MLP kernels read every
    # accumulator back on the vector ALU; no accumulator-register copies)
    ("kd_mlp.hip", True, ["-mllvm", "-amdgpu-mfma-vgpr-form"]),
    ("kd_model.cpp", True, []),
    ("kd_batch.cpp", True, []),
    ("kd_autotune.cpp", True, []),
    ("kd_noalloc.hip", True, []),
    ("kd_build_gpu.hip", True, []),
    ("kd_range_all.hip", True, []),
    ("kd_range_packet.hip", True, []),
]

COMMON = ["-O3", "-std=c++17", "-fPIC", "-ffp-contract=off", "-fno-fast-math", "-Wall",
          "-Wno-unused-function", "-I", os.path.join(ROOT, "include")]
DEVICE = ["--offload-arch=gfx950", "-fno-gpu-flush-denormals-to-zero", "-fno-gpu-rdc",
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]

# Kernels that keep a value of the wave in its lanes (a stack, a list), some of
# which a divergent block leaves inactive.  The register allocator may move such
# a value inside such a block, which loses it there: seen with accumulator
# registers (a walk that never ends), and spills are stored the same way.  A
# build in which one of these kernels has either is refused.
LANE_STATE = ("kd_packet.hip", "kd_range_packet.hip", "kd_wave.hip")
RESOURCES = "-Rpass-analysis=kernel-resource-usage"


def check_lane_state(remarks: str) -> int:
    """Number of kernels in the compiler's resource remarks; raises for one with
    accumulator registers or spilled vector registers."""
    kernel, n = "", 0
    for name, value in re.findall(r"remark: +(Function Name|AGPRs|VGPRs Spill): (\S+)", remarks):
        if name == "Function Name":
            kernel = value
            n += 1
        elif value != "0":
            raise RuntimeError(f"{kernel}: {name} {value}; values kept in inactive lanes would be lost")
    if n == 0:
        raise RuntimeError("no resource remarks from the compiler")
    return n


def _compile(src: str, is_hip: bool, extra: list) -> str:
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *COMMON]
    if is_hip:
        cmd += ["-x", "hip", *DEVICE, *extra]
        if src in LANE_STATE:
            cmd += [RESOURCES]
    cmd += ["-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"compile failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    err = r.stderr
    if src in LANE_STATE:
        try:
            check_lane_state(err)
        except RuntimeError:
            os.remove(obj)
            raise
        # each remark, the source line it quotes and the caret below
        err = re.sub(r"^.*remark: .*\n(?: *\d* \|.*\n)*", "", err, flags=re.M)
    if err.strip():
        # host-pass warnings about the packed-fp32 feature are expected
        lines = [ln for ln in err.splitlines() if "packed-fp32-ops" not in ln]
        if any(ln.strip() for ln in lines):
            sys.stderr.write("\n".join(lines) + "\n")
    return obj


def build(verbose: bool = True) -> str:
    os.makedirs(BUILD, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(lambda s: _compile(*s), SOURCES))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", tmp, *objs, "-lpthread"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB}")
    return LIB


def clean() -> None:
    shutil.rmtree(BUILD, ignore_errors=True)


if __name__ == "__main__":
    build()
