"""Builds librnnd.so (the C-ABI library of include/rnnd.h) in-tree with hipcc for gfx950."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "librnnd.so")
SOURCES = [os.path.join(CSRC, n + ".hip") for n in ("rnnd", "scan_float", "scan_f32", "search")]

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",   # no packed-fp32 VALU ops
    "-mllvm", "-amdgpu-mfma-vgpr-form",     # MFMA accumulators stay in VGPRs: no AGPR round trips in loops
    "-ffp-contract=off", "-Wall", "-Wno-unused-command-line-argument",
]


def _run(cmd):
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    return r.returncode, "\n".join(l for l in r.stdout.splitlines() if "packed-fp32-ops" not in l)


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = "%s.tmp.%d" % (LIB, os.getpid())
    objs = ["%s.%d.o" % (tmp, i) for i in range(len(SOURCES))]
    steps = [[hipcc] + FLAGS + ["-c", "-o", o, s] for o, s in zip(objs, SOURCES)]
    link = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs
    try:
        with ThreadPoolExecutor(len(steps)) as pool:      # one compiler per source
            done = list(pool.map(_run, steps))
        if all(rc == 0 for rc, _ in done):
            done.append(_run(link))
        for (rc, out), cmd in zip(done, steps + [link]):
            if verbose:
                print(" ".join(cmd), flush=True)
            if out.strip() and (verbose or rc):
                (sys.stderr if rc else sys.stdout).write(out + "\n")
        if any(rc for rc, _ in done):
            raise RuntimeError("hipcc failed building librnnd.so")
        os.replace(tmp, LIB)
    finally:
        for f in objs + [tmp]:
            if os.path.exists(f):
                os.remove(f)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
