"""Builds libodma.so (host allocator + gfx950 kernels) in-tree with hipcc."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libodma.so")
# development aids, built beside the library: a timing build whose waves stamp a clock (stream_timeline.py reads it;
# only the bf16 / head_dim 128 decode kernels) and a stand-alone read probe in the attention kernel's launch shape
TIMELINE_LIB = os.path.join(HERE, "libodma_timeline.so")
DEPTH_PROBE = os.path.join(HERE, "read_depth_probe")
# translation units with kernels: (csrc/<source>.hip, object, defines), the one that the timing build replaces first
DEVICE_UNITS = [("odma_stream", f"odma_stream_{f}_{p}", [f"-DODMA_STREAM_FMT={f}", f"-DODMA_STREAM_PLAN={p}"])
                for f in (0, 1, 2) for p in ("false", "true")]
DEVICE_UNITS += [(f"odma_wide_{t}", f"odma_wide_{t}_{p}", [f"-DODMA_STREAM_PLAN={p}"]) for t in ("f32", "bf16") for p in ("false", "true")]
DEVICE_UNITS += [("odma_prefill", "odma_prefill", []), ("odma_device", "odma_device", [])]

HIP_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-fPIC", "-std=c++17",
    # packed fp32 forms are switched off for every kernel in this library
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]
# the allocator's one floating-point helper must round exactly as written
HOST_FLAGS = ["-O2", "-fPIC", "-std=c++17", "-pthread", "-ffp-contract=off", "-Wall", "-Wextra"]


def _run(cmd):
    print("+", " ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)


def build(verbose: bool = True) -> str:
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    cxx = shutil.which("g++") or shutil.which("c++")
    if not os.path.exists(hipcc) or cxx is None:
        raise RuntimeError("hipcc and g++ are required to build libodma")
    inc = ["-I", os.path.join(ROOT, "include"), "-I", CSRC]
    obj_dir = os.path.join(HERE, "_build")
    os.makedirs(obj_dir, exist_ok=True)
    host_o = os.path.join(obj_dir, "odma_host.o")
    _run([cxx, *HOST_FLAGS, *inc, "-c", os.path.join(CSRC, "odma_host.cpp"), "-o", host_o])
    # the device units are independent: compiled side by side
    first = DEVICE_UNITS[0]
    units = DEVICE_UNITS + [(first[0], "odma_stream_timeline", first[2] + ["-DODMA_DEV_TIMELINE", "-DODMA_DEV_MINIMAL_VARIANTS"])]
    cmds = [[hipcc, *HIP_FLAGS, *defs, *inc, "-c", os.path.join(CSRC, src + ".hip"), "-o", os.path.join(obj_dir, obj + ".o")]
            for src, obj, defs in units]
    with ThreadPoolExecutor(max_workers=min(len(cmds), os.cpu_count() or 1, 16)) as ex:
        list(ex.map(_run, cmds))
    objs = [os.path.join(obj_dir, obj + ".o") for _, obj, _ in DEVICE_UNITS]
    _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", host_o, *objs, "-pthread", "-o", LIB])
    timeline = [os.path.join(obj_dir, "odma_stream_timeline.o")] + objs[1:]
    _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", host_o, *timeline, "-pthread", "-o", TIMELINE_LIB])
    _run([hipcc, *[f for f in HIP_FLAGS if f != "-fPIC"], os.path.join(CSRC, "read_depth_probe.hip"), "-o", DEPTH_PROBE])
    return LIB


if __name__ == "__main__":
    build()
    sys.exit(0)
