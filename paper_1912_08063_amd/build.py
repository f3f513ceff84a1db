"""Build libfwi.so (HIP, gfx950) in-tree with hipcc.

    python -m paper_1912_08063_amd.build      # or paper_1912_08063_amd.build.build()
"""
import concurrent.futures
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(HERE, "libfwi.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# (source, extra flags, object): the 3-D step kernels, most of the compile
# time, build once per stencil radius, the largest first
KERNELS = [("fwi_step3d.hip", ["-DFWI_STEP3D_M=%d" % m], "fwi_step3d_m%d.o" % m)
           for m in (8, 4, 2, 1)] + [("fwi_step2d.hip", [], "fwi_step2d.o"),
                                     ("fwi_kernels.hip", [], "fwi_common.o")]
HOST = ["fwi_runtime.cpp", "revolve.cpp"]
# packed-fp32 instructions are disabled: hand-written or generated
# v_pk_{add,mul,fma}_f32 are avoided on this target.  Kernel arguments are
# preloaded into scalar registers (0.3 us less per launch of a small grid: 500
# steps of a 168 x 168 one went from 1767 to 1729 us).
DEVICE_FLAGS = ["--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang",
                "-packed-fp32-ops", "-mllvm", "-amdgpu-kernarg-preload-count=16"]
COMMON = ["-O3", "-std=c++17", "-fPIC", "-Wall", "-I", INCLUDE, "-I", CSRC]


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)


def build(verbose=False, out=None, extra=None):
    """Compile every source and link libfwi.so (or `out`).  `extra` (or the
    environment variable FWI_HIPCC_FLAGS) adds compiler flags, e.g. -D options."""
    extra = list(extra or []) + os.environ.get("FWI_HIPCC_FLAGS", "").split()
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    obj = lambda name: os.path.join(objdir, name)
    cmds = [[HIPCC] + COMMON + DEVICE_FLAGS + extra + flags +
            ["-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj(o)]
            for src, flags, o in KERNELS]
    cmds += [[HIPCC] + COMMON +   # host-only C++ (HIP runtime API only)
             ["-x", "c++", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-c",
              os.path.join(CSRC, src), "-o", obj(src + ".o")] for src in HOST]
    jobs = int(os.environ.get("MAX_JOBS", min(8, os.cpu_count() or 1)))
    with concurrent.futures.ThreadPoolExecutor(max(1, jobs)) as pool:
        list(pool.map(lambda c: _run(c, verbose), cmds))
    # one object with every kernel, which other builds of the host code link
    kernels = obj("fwi_kernels.hip.o")
    _run(["ld", "-r", "-o", kernels] + [obj(o) for _, _, o in KERNELS], verbose)
    lib = out or LIB
    tmp = lib + ".tmp"
    _run([HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", tmp, kernels] +
         [obj(src + ".o") for src in HOST], verbose)
    os.replace(tmp, lib)
    return lib


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
