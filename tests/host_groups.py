"""Builds and loads tests/host_groups.hip: the group kernels' index and
dispatch rules, compiled for the host from the library's own headers."""
import ctypes
import functools
import os
import subprocess
import tempfile

import numpy as np

import paper_2310_11960_amd as F

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = "/opt/rocm/bin/hipcc"
STAGED, GROUPS, STREAM, PAIRS = 1, 2, 4, 8


@functools.lru_cache(maxsize=1)
def library():
    with tempfile.TemporaryDirectory() as d:
        so = os.path.join(d, "host_groups.so")
        cmd = [HIPCC, "-O1", "-std=c++17", "-fPIC", "-shared", "--cuda-host-only", "--offload-arch=gfx950",
               "-Wno-unused-function", "-I", os.path.join(ROOT, "include"),
               "-I", os.path.join(ROOT, "paper_2310_11960_amd", "csrc"),
               os.path.join(ROOT, "tests", "host_groups.hip"), "-Xlinker", F.library()._name, "-o", so,
               "-Wl,-rpath," + os.path.dirname(F.library()._name)]
        r = subprocess.run(cmd, capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-3000:]
        return ctypes.CDLL(so)


def plan_values(op):
    """fma_plan_params of an FMA object, as the int64 array that it writes."""
    cnt = ctypes.c_int32()
    buf = (ctypes.c_int64 * 1024)()
    F._check(F.library().fma_plan_params(op.handle, buf, 1024, ctypes.byref(cnt)))
    return np.frombuffer(buf, dtype=np.int64, count=cnt.value).copy()


def _ptr(v):
    return v.ctypes.data_as(ctypes.POINTER(ctypes.c_int64))


def attend_kernels(v):
    return library().host_attend_kernels(_ptr(v))


def groups_win(v, cus=256):
    return bool(library().host_groups_win(_ptr(v), cus))
