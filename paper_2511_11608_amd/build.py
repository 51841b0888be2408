"""Build libslicer.so (hand-written HIP for gfx950) in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libslicer.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# -ffp-contract=off: the codec's fp32 steps are single IEEE operations (no fused multiply-add);
# packed-fp32 instructions are kept out of the generated code.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wall", "-Wno-unused-function"]


def sources():
    return [os.path.join(CSRC, f) for f in sorted(os.listdir(CSRC)) if f.endswith(".hip")]


def build(verbose: bool = False) -> str:
    """One object per translation unit, compiled in parallel (the row kernels are instantiated many times), then one link."""
    with tempfile.TemporaryDirectory() as tmp:
        units = [(src, os.path.join(tmp, os.path.basename(src) + ".o")) for src in sources()]

        def run(cmd):
            if verbose:
                print(" ".join(cmd))
            subprocess.run(cmd, check=True)

        with ThreadPoolExecutor(max_workers=int(os.environ.get("MAX_JOBS", os.cpu_count() or 1))) as ex:
            for job in [ex.submit(run, [HIPCC, *FLAGS, "-c", src, "-o", obj]) for src, obj in units]:
                job.result()
        run([HIPCC, "--offload-arch=gfx950", "-fPIC", "-shared", *[obj for _, obj in units], "-o", LIB])
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
