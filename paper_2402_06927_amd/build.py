"""Compile the gfx950 HIP library ``libsch.so`` in place (hipcc)."""
from __future__ import annotations

import glob
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "libsch.so")
SOURCES = sorted(glob.glob(os.path.join(HERE, "csrc", "*.hip")))

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++20", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = LIB + ".tmp%d" % os.getpid()
    objects, jobs = [], []
    try:
        for src in SOURCES:  # side by side: a file takes a minute or two
            obj = "%s.%s.o" % (tmp, os.path.basename(src))
            cmd = [hipcc, *HIPCC_FLAGS, "-I", os.path.join(ROOT, "include"),
                   "-I", os.path.join(HERE, "csrc"), "-c", src, "-o", obj]
            if verbose:
                print(" ".join(cmd), file=sys.stderr)
            objects.append(obj)
            jobs.append(subprocess.Popen(cmd))
        codes = [j.wait() for j in jobs]
        for job, code in zip(jobs, codes):
            if code:
                raise subprocess.CalledProcessError(code, job.args)
        subprocess.run([hipcc, "--offload-arch=gfx950", "-shared", *objects, "-o", tmp],
                       check=True)
        os.replace(tmp, LIB)
    finally:
        for obj in objects:
            if os.path.exists(obj):
                os.remove(obj)
    return LIB


def sources_newer_than_lib() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    deps = glob.glob(os.path.join(HERE, "csrc", "*")) + [os.path.join(ROOT, "include", "sch.h")]
    return any(os.path.getmtime(d) > t for d in deps)


if __name__ == "__main__":
    print(build(verbose=True))
