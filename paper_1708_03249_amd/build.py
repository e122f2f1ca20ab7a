"""Build libhhlb.so (HIP for gfx950) in-tree with hipcc.

Run as ``python -m paper_1708_03249_amd.build`` or through
``__graft_entry__.build()``.  Cross-compiles without a GPU.
"""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libhhlb.so")
ARCH = os.environ.get("HHLB_OFFLOAD_ARCH", "gfx950")

HIP_FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
    # packed FP32 instructions stay off (see the design notes)
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-ffp-contract=fast", "-fno-fast-math",
]


def _run(cmd):
    print("+", " ".join(cmd), flush=True)
    subprocess.check_call(cmd)


SOURCES = ("tables.cpp", "hhlb_api.hip", "kernels_fp64.hip", "kernels_mixed_f32.hip",
           "kernels_mixed_bf16.hip", "kernels_mixed_f16.hip", "kernels_large.hip", "kernels_multi.hip",
           "kernels_multi_n3.hip", "kernels_multi_n7.hip", "kernels_multi_n20.hip", "kernels_classes.hip")

# per-source extra flags: the step kernels loop over the stages with most of the
# register file holding the state, and constants moved ahead of that loop
# would only spill (Q = 8: 6 registers spilled instead of 49, Q = 16: 23 instead of 106)
SOURCE_FLAGS = {f: ["-mllvm", "-disable-machine-licm"] for f in (
    "kernels_fp64.hip", "kernels_classes.hip", "kernels_mixed_f32.hip", "kernels_mixed_bf16.hip", "kernels_mixed_f16.hip",
    "kernels_multi_n3.hip", "kernels_multi_n7.hip", "kernels_multi_n20.hip")}


def build(verbose: bool = True, out: str | None = None, defines=()) -> str:
    """Compile libhhlb.so (or `out`); `defines` are extra -D tuning switches.
    The translation units compile in parallel."""
    from concurrent.futures import ThreadPoolExecutor
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objdir = os.path.join(HERE, "_build" + ("_" + "_".join(defines) if defines else ""))
    os.makedirs(objdir, exist_ok=True)
    cmds, objs = [], []
    for src in SOURCES:
        obj = os.path.join(objdir, src + ".o")
        if src.endswith(".cpp"):  # host-only code: plain C++ compiler
            cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-c",
                   os.path.join(CSRC, src), "-o", obj]
        else:
            cmd = [hipcc] + HIP_FLAGS + SOURCE_FLAGS.get(src, []) + [f"-D{d}" for d in defines] + [
                "-c", os.path.join(CSRC, src), "-o", obj]
        cmds.append(cmd)
        objs.append(obj)
    jobs = max(1, min(len(cmds), int(os.environ.get("MAX_JOBS", os.cpu_count() or 1))))
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        list(ex.map(_run, cmds))
    target = out or LIB
    tmp = target + ".tmp"
    _run([hipcc, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp] + objs)
    os.replace(tmp, target)
    return target


if __name__ == "__main__":
    build()
    sys.exit(0)
