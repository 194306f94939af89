"""Build step: compile the HIP sources in csrc/ for gfx950 into libsnip_hip.so and the
native half of the Python binding into _snip_binding.so (in-tree)."""
from __future__ import annotations

import os
import subprocess
from concurrent.futures import ThreadPoolExecutor

_HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(_HERE, "csrc")
LIB = os.path.join(_HERE, "libsnip_hip.so")
BINDING = os.path.join(_HERE, "_snip_binding.so")
MICROBENCH = os.path.join(_HERE, "snip_microbench")
OBJDIR = os.path.join(_HERE, "_build")          # object files (not tracked)
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument"]
# Arguments of a kernel come in scalar registers instead of out of memory: 0.15-0.2 us at the start of a launch (forward of 64 tokens, 7B-shaped,
# eleven launches, 65.7 us -> 63.8, paper recipe 1024 x 1024 x 1024, nine, 51.6 -> 50.2; 1B-shaped block 712 -> 707).  Not for the large GEMM tiles: they run out of scalar
# registers, and two kernels would fetch more spilled ones between the MFMAs.
PRELOAD = ["-mllvm", "-amdgpu-kernarg-preload-count=16"]
NO_PRELOAD = ("gemm_fast.hip",)
SOURCES = ("api.hip", "quant_kernels.hip", "gemm.hip", "gemm_fast.hip", "gemm_small.hip", "optim_kernels.hip", "paper_kernels.hip", "gemm_paper.hip", "gemm_paper_wide.hip")


def binding_command():
    """Host compiler line of the native half of the Python binding (csrc/binding.cpp)."""
    import sysconfig
    import torch
    t = os.path.dirname(torch.__file__)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    return ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f"-I{t}/include",
            f"-I{t}/include/torch/csrc/api/include", f"-I{rocm}/include", f"-I{sysconfig.get_paths()['include']}",
            os.path.join(CSRC, "binding.cpp"), "-o", BINDING, f"-L{t}/lib", "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip", "-ldl"]


def build_library(verbose: bool = False) -> str:
    # one compiler per source file, side by side, then one link
    objs = [os.path.join(OBJDIR, s + ".o") for s in SOURCES]
    os.makedirs(OBJDIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as pool:
        results = list(pool.map(lambda so: subprocess.run(["hipcc"] + FLAGS + ([] if so[0] in NO_PRELOAD else PRELOAD) + ["-fPIC", "-c", "-o", so[1], os.path.join(CSRC, so[0])],
                                                          capture_output=True, text=True), zip(SOURCES, objs)))
    results.append(subprocess.run(binding_command(), capture_output=True, text=True))
    results.append(subprocess.run(["hipcc", "--offload-arch=gfx950", "-fPIC", "-shared", "-o", LIB] + objs, capture_output=True, text=True)
                   if all(r.returncode == 0 for r in results) else results[-1])
    for res in results:
        if verbose or res.returncode != 0:
            print(res.stdout)
            print(res.stderr)
    failed = sorted({os.path.basename(r.args[r.args.index("-o") + 1]) for r in results if r.returncode != 0})
    if failed:
        raise RuntimeError("compiling failed: " + ", ".join(failed))
    # device microbenchmarks (measured roofline denominators), run by `bench.py --microbench`
    cmd = ["hipcc"] + FLAGS + ["-o", MICROBENCH, os.path.join(CSRC, "microbench.hip")]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        print(res.stdout)
        print(res.stderr)
        raise RuntimeError("hipcc failed building snip_microbench")
    return LIB


if __name__ == "__main__":
    print(build_library(verbose=True))
