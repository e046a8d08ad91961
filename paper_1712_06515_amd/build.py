"""Build the gfx950 shared library ``libccr.so`` in-tree with hipcc."""

import os
import subprocess
import sys
import tempfile

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(PKG, "libccr.so")
SOURCES = [os.path.join(CSRC, f) for f in ("ccr_host.cpp", "ccr_kernels.hip", "ccr_lag.hip")]
ARCH = os.environ.get("CCR_OFFLOAD_ARCH", "gfx950")

# Packed FP32 instructions are disabled for all device code (hipcc -O3 would form them from
# float2 arithmetic).
HIP_FLAGS = ["-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def build(out=LIB, extra=(), quiet=True):
    """One hipcc process per source, run together, then the link."""
    flags = [f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function", *HIP_FLAGS,
             "-I", INCLUDE, "-I", CSRC, *extra]

    def check(log, code):
        if code != 0:
            sys.stderr.write(log)
            raise RuntimeError("hipcc build of libccr.so failed")
        if not quiet:
            sys.stderr.write(log)

    with tempfile.TemporaryDirectory(prefix=".build_", dir=PKG) as tmp:
        objs = [os.path.join(tmp, os.path.basename(f) + ".o") for f in SOURCES]
        jobs = [subprocess.Popen(["hipcc", *flags, "-c", f, "-o", o], stdout=subprocess.PIPE,
                                 stderr=subprocess.STDOUT, text=True) for f, o in zip(SOURCES, objs)]
        logs = [j.communicate()[0] for j in jobs]
        for log, j in zip(logs, jobs):
            check(log, j.returncode)
        r = subprocess.run(["hipcc", f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", out + ".tmp"],
                           stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        check(r.stdout, r.returncode)
    os.replace(out + ".tmp", out)
    return out


if __name__ == "__main__":
    print(build(quiet=False))
