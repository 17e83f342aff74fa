"""Build the C-ABI library (csrc/*.hip -> libsbattn.so) for gfx950 with hipcc, and the CPython
module that calls it on torch tensors (csrc/sb_torch.cpp -> _sbtorch.so) with g++.

hipcc cross-compiles without a GPU.  Both are built in-tree, next to this file, so
that they travel with the source tree.
"""
from __future__ import annotations

import glob
import os
import subprocess
import sys
import sysconfig
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libsbattn.so")
EXT = os.path.join(HERE, "_sbtorch.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950",
    # packed fp32 VALU forms are kept out of the generated code on purpose
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # the host pass does not know the packed-fp32 feature name and says so; harmless
    out = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError(f"{cmd[0]} failed:\n" + out)
    if verbose and out.strip():
        print(out)


def _build_ext(obj_dir, verbose):
    """The torch-facing CPython module, plain C++: torch's headers, no device code."""
    import torch
    from torch.utils import cpp_extension
    obj = os.path.join(obj_dir, "sb_torch.o")
    rocm = os.path.dirname(os.path.dirname(HIPCC))
    _run(["g++", "-O2", "-std=c++17", "-fPIC", "-Wall", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
          f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}",
          *[f"-isystem{p}" for p in (*cpp_extension.include_paths(), os.path.join(rocm, "include"),
                                    sysconfig.get_paths()["include"])],
          "-c", os.path.join(CSRC, "sb_torch.cpp"), "-o", obj], verbose)
    return obj


def build(verbose: bool = False, extra=()) -> str:
    """Compile every kernel source and link libsbattn.so, then the module that calls it on torch
    tensors.  Always recompiles."""
    import torch
    torch_lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    with tempfile.TemporaryDirectory() as tmp, ThreadPoolExecutor(max_workers=8) as pool:
        def compile_one(src):
            obj = os.path.join(tmp, os.path.basename(src) + ".o")
            _run([HIPCC, *FLAGS, *extra, "-c", src, "-o", obj], verbose)
            return obj
        ext = pool.submit(_build_ext, tmp, verbose)
        objs = list(pool.map(compile_one, sources()))
        _run([HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", LIB, *objs], verbose)
        _run(["g++", "-shared", "-o", EXT, ext.result(), f"-L{HERE}", "-l:libsbattn.so", "-Wl,-rpath,$ORIGIN", f"-L{torch_lib}",
              "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_hip", "-ltorch", "-ltorch_python"], verbose)
    return LIB


def is_built() -> bool:
    if not (os.path.exists(LIB) and os.path.exists(EXT)):
        return False
    t = min(os.path.getmtime(LIB), os.path.getmtime(EXT))
    deps = sources() + glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(CSRC, "*.cpp")) + \
        [os.path.join(os.path.dirname(HERE), "include", "sb_attn.h")]
    return all(os.path.getmtime(s) <= t for s in deps)


if __name__ == "__main__":
    print(build(verbose=True, extra=sys.argv[1:]))
