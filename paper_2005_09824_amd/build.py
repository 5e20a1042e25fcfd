"""Builds liblfmmi.so (HIP kernels + C ABI) for gfx950, in-tree."""
from __future__ import annotations

import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "liblfmmi.so")
SOURCES = ["kernels.hip", "line.hip", "hybrid.hip", "api.cpp", "pack.cpp"]
HEADERS = ["kernels.h", "device.h", "pack.h", "microbench.hip", os.path.join("..", "..", "include", "lfmmi.h")]

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # scalar fp32 only: no packed-fp32 instructions from the auto-vectoriser
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # private arrays stay out of LDS: kernels here address LDS by absolute offsets
    "-mllvm", "-disable-promote-alloca-to-lds",
    "-Wall", "-Wno-unused-command-line-argument",
]


def is_stale():
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    deps = [os.path.join(CSRC, s) for s in SOURCES + HEADERS] + [os.path.abspath(__file__)]
    return any(os.path.getmtime(d) > t for d in deps)


MICROBENCH = os.path.join(HERE, "lfmmi_microbench")


def microbench_command(hipcc):
    flags = [f for f in FLAGS if f not in ("-fPIC", "-shared")]
    return [hipcc] + flags + ["-o", MICROBENCH, os.path.join(CSRC, "microbench.hip")]


def build(force=True, extra_flags=()):
    """Compile with hipcc (cross-compiles without a GPU): the library, and the
    microbenchmark program behind the roofline peaks."""
    if not force and not is_stale():
        return LIB
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    # every source on its own, side by side: most of the time goes into the kernels' variants
    out = os.path.join(HERE, "_build")
    os.makedirs(out, exist_ok=True)
    objects = [os.path.join(out, src + ".o") for src in SOURCES]
    compile_flags = [f for f in FLAGS if f != "-shared"] + list(extra_flags)
    cmds = [[hipcc] + compile_flags + ["-c", "-o", obj, os.path.join(CSRC, src)]
            for src, obj in zip(SOURCES, objects)]
    cmds.append(microbench_command(hipcc))
    jobs = [subprocess.Popen(c) for c in cmds]
    codes = [j.wait() for j in jobs]
    for code, cmd in zip(codes, cmds):
        if code:
            raise subprocess.CalledProcessError(code, cmd)
    subprocess.check_call([hipcc] + FLAGS + ["-o", LIB] + objects)
    return LIB


if __name__ == "__main__":
    print(build())
