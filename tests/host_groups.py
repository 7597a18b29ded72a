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
ATTEND, ATTEND_128, QUERY, KEY = 0, 1, 2, 3


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


def plan_values(P):
    """The int64 values of a plan (a dict as fma_plan_params returns it)."""
    v = [P[x] for x in F.PLAN_PARAM_NAMES]
    for e in P["sets"]:
        v += [e[x] for x in F.SET_PARAM_NAMES]
    return np.array(v, dtype=np.int64)


def _ptr(v):
    return v.ctypes.data_as(ctypes.POINTER(ctypes.c_int64))


def attend_kernels(v):
    return library().host_attend_kernels(_ptr(v))


def groups_win(v, cus=256):
    return bool(library().host_groups_win(_ptr(v), cus))


def group_count(v):
    fn = library().host_group_count
    fn.restype = ctypes.c_int64
    return fn(_ptr(v))


def group_walk(v, kind, g, wave):
    """kind: ATTEND, ATTEND_128 (head dim 128), QUERY or KEY (backward passes)."""
    out = np.empty(38 + 2304, dtype=np.int64)   # a window of nine cells of 16 x 16
    library().host_group_walk(_ptr(v), kind, g, wave, _ptr(out))
    return dict(active=bool(out[0]), blk=int(out[1]), diag=int(out[3]), lo=int(out[4]), hi=int(out[5]),
                own=out[6:38].copy(), rows=out[38:38 + int(out[2])].copy())


def group_lists(v, per_level, g, wave):
    out = np.empty(5 + 2 * 2048, dtype=np.int64)
    library().host_group_lists(_ptr(v), int(per_level), g, wave, _ptr(out))
    n = int(out[3])
    t = out[5:5 + 2 * n].reshape(n, 2)
    return dict(npiece=int(out[0]), pc0=int(out[1]), npc=int(out[2]), rows=n, blk=int(out[4]), crow=t[:, 0].copy(),
                seen=t[:, 1].astype(bool))


def sibling_group(v, grp):
    gslot = library().host_sibling_slots(_ptr(v))
    out = np.empty(3 + 2 * gslot + 34 * 32, dtype=np.int64)   # at most 4 cells of 8 chunks
    library().host_sibling_group(_ptr(v), grp, _ptr(out))
    nchunk = int(out[2])
    slots = out[3:3 + 2 * gslot].reshape(gslot, 2)
    ch = out[3 + 2 * gslot:3 + 2 * gslot + 34 * nchunk].reshape(nchunk, 34)
    return dict(cx0=int(out[0]), cy0=int(out[1]), rows=slots[:, 0].copy(), masks=slots[:, 1].copy(),
                blocks=ch[:, :2].copy(), tokens=ch[:, 2:].copy())
