"""Builds librnngraph.so (HIP kernels + host planner + C ABI) for gfx950 with hipcc, in-tree."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "librnngraph.so")
SOURCES = ["analyse.cpp", "plan.cpp", "api.cpp", "jit.cpp", "gemm.hip", "elementwise.hip", "step.hip", "static_large.hip"]
EMBEDDED = ["program.h", "step_layout.h", "step_device.h"]   # headers handed to hiprtc at run time
FLAGS = ["-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950", "-munsafe-fp-atomics",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wall", "-Wno-unused-function"]


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objs = []
    procs = []
    os.makedirs(os.path.join(HERE, "_build"), exist_ok=True)
    with open(os.path.join(HERE, "_build", "embedded_sources.h"), "w") as f:
        f.write("// generated by build.py: header texts for the run-time compiler\n#pragma once\n")
        for name in EMBEDDED:
            text = open(os.path.join(CSRC, name)).read()
            assert ")RNNGSRC\"" not in text
            f.write(f"static const char* const RNNG_SRC_{name.replace('.', '_')} = R\"RNNGSRC({text})RNNGSRC\";\n")
    for src in SOURCES:
        obj = os.path.join(HERE, "_build", src + ".o")
        cmd = [hipcc, *FLAGS, "-I", os.path.join(HERE, "_build"), "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    failed = False
    for src, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode != 0:
            failed = True
            print(f"[build] {src} FAILED\n{out}", file=sys.stderr)
        elif out.strip() and verbose:
            print(out)
    if failed:
        raise RuntimeError("hipcc failed")
    cmd = [hipcc, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", LIB, *objs, "-ldl"]
    subprocess.run(cmd, check=True)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
