"""Build the native libraries in-tree: the HIP library (gfx950) and the input generator."""

from __future__ import annotations

import os
import shutil
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libtamm_mi.so")
SOURCES = ["capi_core.cpp", "plan.cpp", "denominator.cpp", "addop.cpp", "sched.cpp", "cholesky.cpp", "kernels.hip", "kernels_mixed.hip",
           "kernels_elem.hip", "diag.hip", "noalloc.hip"]
HIPCC_FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-shared",
    # packed FP32 instructions are never generated (see the design notes on gfx950 hazards)
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # MFMA accumulators in architectural VGPRs: without it the loop-carried accumulators are
    # copied between VGPRs and AGPRs on every K chunk
    "-mllvm", "-amdgpu-mfma-vgpr-form",
    "-I" + os.path.join(ROOT, "include"),
]


def hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if c and os.path.exists(c):
            return c
    raise RuntimeError("hipcc not found; the HIP library cannot be built")


# kernels.hip compiles in parts (part 0: everything but the float64 contraction kernels), so that
# its many template instances build side by side
F64_PARTS = 6


def units():
    """(source, extra flags, object name) of every compilation; the longest first."""
    out = []
    for s in SOURCES:
        for part in range(F64_PARTS if s == "kernels.hip" else 1):
            flags = ["-DTAMM_F64_PART=%d" % part] if s == "kernels.hip" else []
            out.append((os.path.join(CSRC, s), flags, "%s.%d.o" % (s, part)))
    return sorted(out, key=lambda u: not (u[1] and u[1] != ["-DTAMM_F64_PART=0"]))


def build_hip(verbose: bool = False) -> str:
    """Compile every source to an object in parallel, then link the shared library in place."""
    import tempfile
    from concurrent.futures import ThreadPoolExecutor

    compile_flags = [f for f in HIPCC_FLAGS if f != "-shared"]
    with tempfile.TemporaryDirectory(prefix="tamm_build_") as tmpdir:
        objs = [os.path.join(tmpdir, name) for _, _, name in units()]
        cmds = [[hipcc()] + compile_flags + flags + ["-c", "-o", obj, src] for (src, flags, _), obj in zip(units(), objs)]
        if verbose:
            for c in cmds:
                print(" ".join(c), flush=True)
        with ThreadPoolExecutor(max_workers=min(len(cmds), os.cpu_count() or 1)) as ex:
            for f in [ex.submit(subprocess.check_call, c) for c in cmds]:
                f.result()
        tmp = LIB + ".tmp%d" % os.getpid()
        link = [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs
        if verbose:
            print(" ".join(link), flush=True)
        subprocess.check_call(link)
        os.replace(tmp, LIB)
    return LIB


def build_all(verbose: bool = False):
    from .synth import build_library

    build_library(force=True)
    return build_hip(verbose)


if __name__ == "__main__":
    build_all(verbose=True)
