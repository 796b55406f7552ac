"""Runs a script against libpsdf.so on the host runtime of host/fake_hip.cpp:
plans are created, calls are validated and dispatched, kernels are listed
instead of run.  The script runs in a process of its own, without torch."""
import json
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = '''
import ctypes, json, sys, types
sys.path.insert(0, {root!r})
sys.modules["torch"] = types.ModuleType("torch")   # its HIP runtime must stay out
hip = ctypes.CDLL({shim!r}, mode=ctypes.RTLD_GLOBAL)
hip.fake_limit.argtypes = [ctypes.c_size_t]
hip.fake_fail_malloc.argtypes = [ctypes.c_long]
hip.fake_used.restype = ctypes.c_size_t
hip.fake_launches.restype = ctypes.c_char_p
import numpy as np
from paper_2607_04310_amd import _lib
lib = _lib.lib()
ONE = ctypes.c_void_p(4096)          # stands for any device pointer
HEX = [[0.5, 0.0], [0.25, 0.43], [-0.25, 0.43], [-0.5, 0.0], [-0.25, -0.43], [0.25, -0.43]]


def launches():
    """[(kernel, grid x, grid y, work-group), ...] since the last call."""
    out = [(r[0], *map(int, r[1:])) for r in
           (line.split() for line in hip.fake_launches().decode().splitlines())]
    hip.fake_clear()
    return out


def kernels(words=("cull_list", "cull_stage_kernel", "cull_stage_edges", "cull_main", "stage_batch",
                   "batch_kernel", "screen_bound", "main_staged", "main_kernel", "small_quad",
                   "small_kernel")):
    """The launches by the kernels' names (mangled names hold them)."""
    return [next((w for w in words if w in k[0]), "other") for k in launches()]


def params(eps=1e-12, eps_sat=1e-6, eta=1000.0):
    return _lib.PsdfParams(eps, eps_sat, eta)


def plan(insts, mbar=4, par=None, flags=0):
    """(code, plan) of instances (footprint, N, M, E)."""
    fps = np.concatenate([np.asarray(i[0], np.float32) for i in insts])
    desc, at = [], [0, 0, 0, 0]
    for fp, N, M, E in insts:
        desc.append(_lib.PsdfBatchDesc(at[0], len(fp), at[1], N, at[2], E, at[3], M))
        at = [at[0] + len(fp), at[1] + N, at[2] + E, at[3] + M + 1]
    p = ctypes.c_void_p()
    par = par or params()
    rc = lib.psdf_batch_plan_create(ctypes.byref(p), (_lib.PsdfBatchDesc * len(desc))(*desc), len(desc),
                                    fps.ctypes.data_as(ctypes.c_void_p), mbar, ctypes.byref(par), flags)
    return rc, p


def run(p):
    assert lib.psdf_batch(p, *[ONE] * 11, None) == 0, lib.psdf_last_error()
    return kernels()


def autotune(p):
    assert lib.psdf_batch_autotune(p, *[ONE] * 11, None, None) == 0
    launches()


def bound(p):
    assert lib.psdf_batch_screened_bound(p, *[ONE] * 11, None, None, None, None) == 0
    return kernels()


def stage(p):
    rc = lib.psdf_batch_stage(p, *[ONE] * 5, None)
    return rc, kernels()


def plain(fp, N, M, mbar=4, par=None):
    """Kernels of a psdf_eval of N stages against M obstacles."""
    fp = np.ascontiguousarray(fp, np.float32)
    e = _lib.PsdfEdges(4096, 4096, 4096, 4096, 4096, M, M, mbar)
    par = par or params()
    rc = lib.psdf_eval(fp.ctypes.data_as(ctypes.c_void_p), len(fp), ONE, N, ctypes.byref(e),
                       ctypes.byref(par), ONE, ONE, ONE, ONE, ONE, 1 << 50, None)
    assert rc == 0, lib.psdf_last_error()
    return kernels()


def emit(x):
    print("RESULT " + json.dumps(x))
'''

_shim = None


def script(body, tmp_path_factory, env=None):
    """The object that `body` passes to emit()."""
    global _shim
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    if _shim is None:
        _shim = str(tmp_path_factory.mktemp("fake_hip") / "libfakehip.so")
        subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared",
                        os.path.join(HERE, "host", "fake_hip.cpp"), "-o", _shim], check=True,
                       capture_output=True, timeout=300)
    code = PRELUDE.format(root=ROOT, shim=_shim) + body
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=300,
                       env=dict(os.environ, **(env or {})))
    assert r.returncode == 0, (r.returncode, r.stdout[-500:], r.stderr[-2000:])
    return json.loads(r.stdout.rsplit("RESULT ", 1)[1])
