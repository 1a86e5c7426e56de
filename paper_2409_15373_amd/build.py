"""Build libjfa.so in-tree with hipcc for gfx950 (cross-compiles without a GPU), and beside it the C++ autograd nodes (host code against
the installed torch; the library does without them, and where they cannot be built that is said and the library is built all the same).

    python -m paper_2409_15373_amd.build [--force]
"""
from __future__ import annotations

import concurrent.futures
import glob
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libjfa.so")
NATIVE_SRC = os.path.join(CSRC, "jfa_autograd.cpp")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc", "-Wall", "-Wno-unused-function",
    # packed fp32 VALU ops stay off (some of their forms have produced wrong results on these machines)
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # the global -> LDS copies are written as inline asm that sets m0, a register the compiler reserves: the clobber is declared on purpose
    "-Wno-inline-asm",
]


def _stale(target: str, deps) -> bool:
    if not os.path.exists(target):
        return True
    t = os.path.getmtime(target)
    return any(os.path.getmtime(d) > t for d in deps)


def _compile(src: str, force: bool, extra) -> str:
    obj = os.path.join(OBJ, os.path.basename(src) + ".o")
    headers = glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(HERE, "..", "include", "*.h"))
    if force or _stale(obj, [src] + headers):
        cmd = [HIPCC] + FLAGS + list(extra) + ["-c", src, "-o", obj]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
        warn = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l and l.strip())
        if "warning" in warn:
            sys.stderr.write(warn + "\n")
    return obj


def native_path(torch_version: str) -> str:
    """The C++ autograd nodes' file: it fits one torch and one Python, whose versions its name carries."""
    return os.path.join(HERE, f"_native.torch-{torch_version}.{sysconfig.get_config_var('SOABI')}.so")


def _build_native(force: bool) -> None:
    import torch
    from torch.utils import cpp_extension
    target = native_path(torch.__version__)
    if not (force or _stale(target, [NATIVE_SRC])):
        return
    if os.path.exists(target):
        os.remove(target)   # not to be left behind by a build that fails
    lib_dir = os.path.join(os.path.dirname(torch.__file__), "lib")
    includes = cpp_extension.include_paths() + [os.path.join(os.path.dirname(os.path.dirname(HIPCC)), "include"), sysconfig.get_paths()["include"]]
    tmp = target + ".tmp"
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM",
           "-DTORCH_EXTENSION_NAME=_native", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           *(f"-isystem{i}" for i in includes), NATIVE_SRC, "-o", tmp, f"-L{lib_dir}", "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch", "-ltorch_python"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"{cmd[0]} failed for {NATIVE_SRC}:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, target)


def build(force: bool = False, extra_flags=()) -> str:
    os.makedirs(OBJ, exist_ok=True)
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        native = ex.submit(_build_native, force)
        objs = list(ex.map(lambda s: _compile(s, force, extra_flags), srcs))
    if force or _stale(LIB, objs):
        tmp = LIB + ".tmp"
        r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs,
                           capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
        os.replace(tmp, LIB)
    try:
        native.result()
    except Exception as e:   # no torch, no headers, no compiler
        sys.stderr.write(f"The C++ autograd nodes are not built, the Python functions of autograd.py do their work more slowly:\n{e}\n")
    return LIB


if __name__ == "__main__":
    print(build(force="--force" in sys.argv))
