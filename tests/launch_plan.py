"""Builds tests/host/plan.cpp against the library's host code and binds it."""
import ctypes
import functools
import os
import subprocess

from paper_2007_01277_amd import build as B
from paper_2007_01277_amd import hfuse as H

SRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "host", "plan.cpp")
SO = os.path.join(B.BUILD, "plan.so")


@functools.lru_cache(maxsize=1)
def lib():
    H.lib()
    os.makedirs(B.BUILD, exist_ok=True)
    cmd = [B.HIPCC] + B.FLAGS + ["-x", "hip", "--offload-host-only", "-shared", SRC, "-x", "none", B.LIB,
                                 f"-Wl,-rpath,{B.PKG}", "-o", SO]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    L = ctypes.CDLL(SO)
    t = ctypes.POINTER(H.hf_task)
    for name, res, args in (("plan_wgs", ctypes.c_uint32, [t] + [ctypes.c_int] * 5),
                            ("plan_useful", ctypes.c_int64, [t, ctypes.c_int]),
                            ("plan_own_scratch", ctypes.c_int64, [t]),
                            ("plan_slot", ctypes.c_int64, [ctypes.c_int64]), ("plan_upsample_path", ctypes.c_int, [t])):
        f = getattr(L, name)
        f.restype, f.argtypes = res, args
    return L


def task(kind, shape=(0, 0, 0, 0), p=(), misalign=0, idx=False, scratch=False):
    """A descriptor whose pointers are never followed; `misalign` bytes past a
    line for the image buffers."""
    t = H.hf_task()
    t.kind = kind
    base = 1 << 32
    t.in_, t.out0 = base + misalign, 2 * base + misalign
    t.out1 = 3 * base if kind == H.HF_BN_STATS or idx else None
    t.in1 = 4 * base if kind == H.HF_ETHASH else None
    t.scratch = 5 * base if scratch else None
    t.n, t.c, t.h, t.w = (tuple(shape) + (0, 0, 0))[:4]
    for i, v in enumerate(p):
        t.p[i] = v
    assert H.hf_validate_task(t) == H.HF_OK
    return t


def wgs(t, waves, block, resident, num_cus=256, own=True):
    return lib().plan_wgs(ctypes.byref(t), int(own), waves, block, resident, num_cus)


def useful(t, waves):
    return lib().plan_useful(ctypes.byref(t), waves)


def own_scratch(t):
    return lib().plan_own_scratch(ctypes.byref(t))


def slot(nbytes):
    return lib().plan_slot(nbytes)


def upsample_path(t):
    return lib().plan_upsample_path(ctypes.byref(t))
