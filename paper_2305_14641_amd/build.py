"""Build the HIP library in-tree with hipcc for gfx950.

    python -m paper_2305_14641_amd.build

Every translation unit under csrc/ is compiled to an object file (in
parallel), then linked into ``libqc_hip.so`` next to this file. Device code
is built with packed FP32 instructions disabled.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import re
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
OBJDIR = os.path.join(ROOT, "_build")
LIB = os.path.join(HERE, "libqc_hip.so")

SOURCES = ["qc_kernels.hip", "qc_dense.hip", "qc_bfs_4.hip", "qc_bfs_8.hip", "qc_bfs_16.hip", "qc_bfs_32.hip",
           "qc_bfs_64.hip", "qc_api.cpp", "qc_host.cpp", "qc_timing.cpp", "qc_batch.cpp",
           "qc_server.cpp", "qc_noalloc.hip", "qc_sssp.hip", "qc_real.cpp",
           "qc_count_512.hip", "qc_count_1024.hip", "qc_dist_4.hip", "qc_dist_5.hip", "qc_dist_7.hip",
           "qc_rows.cpp", "qc_search.cpp", "qc_onecall.cpp", "qc_descend.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
COMMON = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall",
          "-I" + INCLUDE, "-I" + CSRC,
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


# Kernels that must keep every scalar register (see qc_count.h).
NO_SCALAR_SPILLS = "k_count"


def scalar_spills(remarks: str) -> dict:
    """Scalar registers spilled per kernel, from the compiler's
    kernel-resource-usage remarks."""
    spills, name = {}, None
    for line in remarks.splitlines():
        m = re.search(r"remark:.*Function Name: (\S+)", line)
        if m:
            name = m.group(1)
        m = re.search(r"remark:.*SGPRs Spill: (\d+)", line)
        if m and name is not None:
            spills[name] = int(m.group(1))
    return spills


def check_spills(src: str, remarks: str) -> None:
    spills = {k: v for k, v in scalar_spills(remarks).items() if NO_SCALAR_SPILLS in k}
    if not spills and src.startswith(("qc_count_", "qc_dist_")):
        raise RuntimeError(f"{src}: no resource remarks of {NO_SCALAR_SPILLS}")
    bad = {k: v for k, v in spills.items() if v}
    if bad:
        raise RuntimeError(f"{src}: scalar registers spilled in {bad}")


def _compile(src: str) -> str:
    path = os.path.join(CSRC, src)
    obj = os.path.join(OBJDIR, src + ".o")
    cmd = [HIPCC] + COMMON + ["-Rpass-analysis=kernel-resource-usage", "-x", "hip", "-c", path, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    check_spills(src, r.stderr)
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(OBJDIR, exist_ok=True)
    srcs = [s for s in SOURCES if os.path.exists(os.path.join(CSRC, s))]
    with cf.ThreadPoolExecutor(max_workers=min(12, len(srcs))) as ex:
        objs = list(ex.map(_compile, srcs))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs + ["-lpthread"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
