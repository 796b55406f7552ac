"""Compile the HIP sources of the package into ``libpsdf.so`` (gfx950), and the
native Python calls into ``_native.so``.

Each translation unit is compiled to an object in parallel, then linked.
Flags: -O3, -ffp-contract=off (every fused multiply-add is explicit in the
source, so all kernels that share the device arithmetic agree bit for bit),
and packed FP32 instructions disabled for the device code.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(HERE, "libpsdf.so")
NATIVE = os.path.join(HERE, "_native.so")
BUILD_DIR = os.path.join(ROOT, "_build")

SOURCES = (["psdf_host.cpp", "psdf_plain.hip", "psdf_batch.hip", "psdf_mlp.hip", "psdf_geom.hip"]
           + [f"psdf_inst_mf{m}.hip" for m in (3, 4, 5, 6, 7, 8, 16)]
           + [f"psdf_batch_mf{m}.hip" for m in (3, 4, 5, 6, 7, 8, 16)]
           + [f"psdf_screen_mf{m}.hip" for m in (3, 4, 5, 6, 7, 8, 16)])

ARCH = os.environ.get("PSDF_OFFLOAD_ARCH", "gfx950")
COMMON = ["-O3", "-std=c++17", "-fPIC", "-ffp-contract=off", f"-I{INCLUDE}", f"-I{CSRC}"]
DEVICE = [f"--offload-arch={ARCH}", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _hipcc():
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    return exe


def _compile(src: str) -> str:
    path = os.path.join(CSRC, src)
    obj = os.path.join(BUILD_DIR, os.path.splitext(src)[0] + ".o")
    cmd = [_hipcc()] + COMMON + DEVICE
    if src.endswith(".hip"):
        cmd += ["-x", "hip"]
    cmd += ["-c", path, "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{res.stderr}")
    return obj


def _compile_native() -> str:
    """Object of the CPython module (host code, against torch's headers)."""
    import sysconfig

    import torch
    from torch.utils import cpp_extension

    obj = os.path.join(BUILD_DIR, "psdf_native.o")
    inc = cpp_extension.include_paths() + [sysconfig.get_paths()["include"],
                                           os.path.join(_rocm(), "include"), INCLUDE]
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__=1",
           "-DUSE_ROCM=1", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           *[f"-isystem{d}" for d in inc], "-c", os.path.join(CSRC, "psdf_native.cpp"), "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"g++ failed for psdf_native.cpp:\n{res.stderr}")
    return obj


def _rocm() -> str:
    return os.path.dirname(os.path.dirname(os.path.realpath(_hipcc())))


def _link_native(obj: str) -> None:
    """_native.so beside libpsdf.so, which it loads from its own folder (the
    file that _lib.py opens: one copy of the library in a process)."""
    from torch.utils import cpp_extension

    tmp = NATIVE + ".tmp"
    cmd = ["g++", "-shared", "-fPIC", obj, "-o", tmp, f"-L{HERE}", "-l:libpsdf.so",
           *[f"-L{d}" for d in cpp_extension.library_paths()], "-lc10", "-lc10_hip", "-ltorch_cpu",
           "-ltorch_python", "-Wl,-rpath,$ORIGIN", "-Wl,--allow-shlib-undefined"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"link of _native.so failed:\n{res.stderr}")
    os.replace(tmp, NATIVE)


def build(jobs: int | None = None) -> str:
    os.makedirs(BUILD_DIR, exist_ok=True)
    jobs = jobs or min(8, len(SOURCES))
    with cf.ThreadPoolExecutor(jobs) as ex:
        native = ex.submit(_compile_native)
        objs = list(ex.map(_compile, SOURCES))
        native_obj = native.result()
    tmp = LIB + ".tmp"
    cmd = [_hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", tmp]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"link failed:\n{res.stderr}")
    os.replace(tmp, LIB)
    _link_native(native_obj)
    return LIB


if __name__ == "__main__":
    print(build())
    sys.exit(0)
