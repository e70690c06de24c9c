"""Build step: compile the HIP sources in csrc/ into libblr.so for gfx950 (cross-compiles without a GPU) and
csrc/host_call.cpp, the native callables of the Python binding, into _host.so."""
from __future__ import annotations

import glob
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(HERE, "libblr.so")
HOST = os.path.join(HERE, "_host.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-shared", "-fPIC",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def sources():
    return sorted(glob.glob(os.path.join(HERE, "csrc", "*.hip")))


def _host_command():
    """g++ command line of the binding's extension module: torch's own C++ headers and libraries, and libblr.so beside it."""
    import shutil
    import sysconfig
    import torch
    t = os.path.dirname(torch.__file__)
    rocm = os.path.dirname(os.path.dirname(os.path.abspath(shutil.which(HIPCC) or HIPCC)))     # (HIPCC may be a bare command name)
    return ["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__=1",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
            "-isystem", os.path.join(t, "include"), "-isystem", os.path.join(t, "include", "torch", "csrc", "api", "include"),
            "-isystem", os.path.join(rocm, "include"), "-isystem", sysconfig.get_paths()["include"],
            os.path.join(HERE, "csrc", "host_call.cpp"), "-o", HOST,
            "-L" + os.path.join(t, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip", "-L" + HERE, "-l:libblr.so", "-Wl,-rpath,$ORIGIN"]


def _run(cmd):
    res = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in res.stderr.splitlines() if noise not in l)
    if res.returncode != 0:
        raise RuntimeError("compilation failed:\n" + " ".join(cmd) + "\n" + err)
    return err


def build_library(verbose: bool = False) -> str:
    """Compile every kernel translation unit (in parallel), link the C-ABI shared library in-tree, then the binding's extension module."""
    import tempfile
    from concurrent.futures import ThreadPoolExecutor
    srcs = sources()
    with tempfile.TemporaryDirectory(prefix="blr_build_") as tmp:
        objs = [os.path.join(tmp, os.path.basename(src) + ".o") for src in srcs]
        compile_flags = [f for f in FLAGS if f != "-shared"]
        with ThreadPoolExecutor(max_workers=min(8, len(srcs))) as pool:
            errs = list(pool.map(lambda so: _run([HIPCC] + compile_flags + ["-c", so[0], "-o", so[1]]), zip(srcs, objs)))
        errs.append(_run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC"] + objs + ["-o", LIB]))
    errs.append(_run(_host_command()))
    if verbose and any(e.strip() for e in errs):
        print("\n".join(e for e in errs if e.strip()))
    return LIB


if __name__ == "__main__":
    print(build_library(verbose=True))
