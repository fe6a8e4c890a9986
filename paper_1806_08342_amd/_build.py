"""Builds libqnn.so (the C-ABI library) from the HIP sources with hipcc for gfx950, and _native.so, the
compiled Python binding on top of it.

Both are built in-tree, next to this file; nothing is compiled at import time.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libqnn.so")
NATIVE = os.path.join(HERE, "_native.so")
# (the ones that take longest first)
SOURCES = ["igemm_bres.hip", "igemm_bres4.hip", "igemm_ring_int8_low.hip", "igemm_ring_int4_low.hip", "igemm.hip", "igemm_shortk.hip", "igemm_shortk4.hip",
           "dwconv.hip", "igemm_ring_int8_high.hip", "igemm_ring_int4_high.hip", "igemm_tiles.hip", "igemm_stem.hip", "igemm_smallk.hip", "igemm_tail.hip",
           "igemm_tile64.hip", "elementwise.hip", "igemm_repack.hip", "host_helpers.hip", "calibrate.hip"]
FLAGS = [
    "-O3",
    "--offload-arch=gfx950",
    "-std=c++17",
    "-fPIC",
    "-Wall",
    # packed-FP32 instructions are switched off for all device code of this library
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def _compile(src: str) -> str:
    obj = os.path.join(CSRC, src.replace(".hip", ".o"))
    cmd = ["hipcc", *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(ln for ln in res.stderr.splitlines() if "packed-fp32-ops" not in ln)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{err}")
    if err.strip():
        print(err)
    return obj


def _compile_binding() -> str:
    """The Python binding is host code only: a plain C++ compilation against torch's headers."""
    from torch.utils import cpp_extension

    obj = os.path.join(CSRC, "binding.o")
    incs = [f"-I{d}" for d in cpp_extension.include_paths("cuda") + [sysconfig.get_paths()["include"]] if os.path.isdir(d)]
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-fPIC", "-Wall", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
                           *incs, "-c", os.path.join(CSRC, "binding.cpp"), "-o", obj])
    return obj


def build_library(verbose: bool = True) -> str:
    """Compile every HIP source for gfx950, link libqnn.so and the Python binding.  Always recompiles."""
    from torch.utils import cpp_extension

    with cf.ThreadPoolExecutor(max_workers=min(8, len(SOURCES) + 1)) as pool:
        binding = pool.submit(_compile_binding)
        objs = list(pool.map(_compile, SOURCES))
        binding_obj = binding.result()
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs])
    torch_lib = cpp_extension.library_paths("cuda")[0]
    subprocess.check_call(["g++", "-shared", "-o", NATIVE, binding_obj, f"-L{HERE}", "-lqnn", f"-L{torch_lib}", "-lc10", "-ltorch_cpu", "-ltorch_python",
                           "-lc10_hip", "-ltorch_hip", "-Wl,-rpath,$ORIGIN"])
    if verbose:
        print(f"built {LIB} and {NATIVE}")
    return LIB


if __name__ == "__main__":
    build_library()
