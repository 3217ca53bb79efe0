"""Builds ``libcgx.so`` (HIP kernels + C ABI) for gfx950 with hipcc, in-tree."""
from __future__ import annotations

import os
import subprocess
import warnings
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libcgx.so")
ARGS = os.path.join(HERE, "_cgx_args.so")
OBJ = os.path.join(HERE, "_build")
# (source, object name, extra flags): the quantize, reduce and fused kernels are built for chunks of 1024 and of 2048 elements
SOURCES = [("cgx_plan.cpp", "cgx_plan", []), ("cgx_api.cpp", "cgx_api", []), ("cgx_adaptive.cpp", "cgx_adaptive", []),
           ("cgx_quantize.hip", "cgx_quantize_g2", ["-DCGX_GROUPS=2"]),
           ("cgx_quantize.hip", "cgx_quantize_g4", ["-DCGX_GROUPS=4"]),
           ("cgx_reduce.hip", "cgx_reduce_g2", ["-DCGX_GROUPS=2"]),
           ("cgx_reduce.hip", "cgx_reduce_g4", ["-DCGX_GROUPS=4"]), ("cgx_fused.hip", "cgx_fused_g2", ["-DCGX_GROUPS=2"]),
           ("cgx_fused.hip", "cgx_fused_g4", ["-DCGX_GROUPS=4"]), ("cgx_wide.hip", "cgx_wide", []),
           ("cgx_stats.hip", "cgx_stats", []),
           ("cgx_probe.hip", "cgx_probe", [])]

# -ffp-contract=off: the code decision is binary32 without fused operations.
# packed-fp32 instructions stay disabled for this target.
# kernarg preload: the dispatcher puts the first 16 dwords of a kernel's arguments into scalar registers, so a
# wave's first scalar load is its tile descriptor (0.5 us per launch of 20 us); firmware without the feature
# runs the loads of the compiler's compatibility prologue instead.
# no machine-level hoisting: every kernel is a loop over tiles that normally runs once or twice, and what the compiler
# moves in front of it (constants of all bit widths' paths) stays in registers across all of them.  Without it the
# binary32 quantizer needs 44 vector registers instead of 63 and spills no scalar ones, the binary16 one 69 instead of
# 84 (decompressing 355 M elements to binary16 in 8 shares: 197 -> 187 us; quantizing them: 162 -> 159 us).
FLAGS = ["-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC", "-ffp-contract=off",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-mllvm", "-amdgpu-kernarg-preload-count=16", "-mllvm", "-disable-machine-licm",
         "-Wall", "-Wno-unused-command-line-argument", "-Wno-unused-function"]


def build(verbose: bool = False, extra=(), jobs: int = 8) -> str:
    """Compiles every source (in parallel: the kernel files take a minute each) and links.  The extension module that
    checks tensors needs g++ and torch's headers besides; without it the library is complete and the binding makes the
    checks in Python, so a failure there is a warning."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(OBJ, exist_ok=True)

    def compile_one(item):
        src, name, flags = item
        obj = os.path.join(OBJ, name + ".o")
        cmd = [hipcc, *FLAGS, *flags, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd))
        subprocess.run(cmd, check=True, cwd=CSRC)
        return obj

    def compile_args():
        # the binding's tensor checks: host code against torch's headers
        import sysconfig

        import torch
        from torch.utils.cpp_extension import include_paths
        libs = os.path.join(os.path.dirname(torch.__file__), "lib")
        cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
               *(f"-I{d}" for d in (*include_paths(), sysconfig.get_paths()["include"])),
               os.path.join(CSRC, "cgx_tensor_args.cpp"), "-o", ARGS, f"-L{libs}", "-ltorch_python", "-ltorch_cpu", "-lc10",
               f"-Wl,-rpath,{libs}"]
        if verbose:
            print(" ".join(cmd))
        subprocess.run(cmd, check=True, cwd=CSRC)

    with ThreadPoolExecutor(max_workers=max(1, min(jobs, len(SOURCES) + 1))) as pool:
        args = pool.submit(compile_args)
        objs = list(pool.map(compile_one, SOURCES))
        failure = args.exception()
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    if verbose:
        print(" ".join(cmd))
    subprocess.run(cmd, check=True, cwd=CSRC)
    if failure is not None:
        if os.path.exists(ARGS):
            os.remove(ARGS)                      # of other sources, or for another torch
        warnings.warn(f"_cgx_args.so was not built: {failure}", RuntimeWarning)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
