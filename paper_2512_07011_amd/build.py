"""Builds libbsfa.so (the HIP kernels and their C ABI) in-tree for gfx950 with hipcc."""
from __future__ import annotations

import os
import subprocess
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libbsfa.so")
# translation units: (source, extra flags).  bsfa_fwd.hip is compiled once per group of kernel instantiations.
FWD_PARTS = 11
UNITS = [("bsfa_fwd.hip", ["-DBSFA_PART=%d" % i]) for i in range(FWD_PARTS)] + \
        [(s, []) for s in ("bsfa_select.hip", "bsfa_probe.hip", "bsfa_api.hip")]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         # accumulators in plain VGPRs: kernels whose LDS leaves room for one wave per SIMD would otherwise be given
         # AGPRs and copy between the two (1.2x slower at 64 and 32 query rows per tile)
         "-mllvm", "-amdgpu-mfma-vgpr-form=1",
         # packed-fp32 VALU forms are kept out of the generated code on this target
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         # the tile copies set M0 in inline asm and list it as clobbered, which clang notes for every
         # instantiation (thousands of identical lines): that one diagnostic is switched off
         "-Wall", "-Wno-unused-function", "-Wno-inline-asm"]


def build_lib(verbose: bool = False, extra_flags=(), lib: str = LIB) -> str:
    """Compile every translation unit (side by side) and link them into ``lib``; returns its path."""
    tmp = lib + ".tmp.%d" % os.getpid()
    objs = ["%s.%d.o" % (tmp, i) for i in range(len(UNITS))]

    def run(cmd):
        r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        out = "\n".join(l for l in r.stdout.splitlines() if "is not a recognized feature for this target" not in l)
        if r.returncode != 0:
            raise RuntimeError("hipcc failed:\n" + " ".join(cmd) + "\n" + out)
        if verbose and out.strip():
            print(out)

    try:
        cmds = [[HIPCC, *FLAGS, *extra_flags, *more, "-c", "-o", obj, os.path.join(CSRC, src)] for (src, more), obj in zip(UNITS, objs)]
        if verbose:
            print("\n".join(" ".join(c) for c in cmds), flush=True)
        with ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as pool:
            list(pool.map(run, cmds))
        run([HIPCC, "--offload-arch=gfx950", "-fPIC", "-shared", "-o", tmp, *objs])
        os.replace(tmp, lib)
    finally:                      # an interrupted or failed build leaves no partial library behind
        for f in [tmp, *objs]:
            if os.path.exists(f):
                os.remove(f)
    return lib


if __name__ == "__main__":
    print(build_lib(verbose=True))
