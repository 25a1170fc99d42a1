"""CPU tests of the library's host code on a stand-in HIP runtime
(host_hip.cpp): ``run(source)`` executes a Python program in a process of its
own in which ``hip`` is the stand-in and ``L`` the library bound to it."""
from __future__ import annotations

import functools
import os
import subprocess
import sys
import tempfile
import textwrap

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes as C, sys
import numpy as np
sys.path.insert(0, {root!r})
hip = C.CDLL({lib!r}, mode=C.RTLD_GLOBAL)
for f in ("host_launches", "host_pinned", "host_recorded"):
    getattr(hip, f).restype = C.c_int64
hip.host_stream.restype = C.c_void_p
hip.host_capture.argtypes = [C.c_void_p, C.c_int]
hip.host_launch.argtypes = [C.c_int64, C.c_void_p]
from paper_2109_12855_amd import sdeliver, workloads as W
L = sdeliver.lib()

def create(cfg, stream=None, build=True):
    h = C.c_void_p()
    c = sdeliver.make_config(cfg)
    assert L.sd_create(C.byref(c), stream, None, 0, C.byref(h)) == 0, L.sd_last_error(h)
    if build:
        assert L.sd_build_connections(h) == 0, L.sd_last_error(h)
    return h

def launches():
    out = np.zeros((hip.host_launches(), 8), np.int64)
    for i in range(len(out)):
        hip.host_launch(i, out[i].ctypes.data)
    return out  # kind (1 persistent, 2 one slice), stream, slices, first tag, lanes

def read(h, n):
    a = [np.zeros(n, np.float32) for _ in range(3)] + [np.zeros(n, np.int32)]
    return L.sd_read_state(h, *[C.c_void_p(x.ctypes.data) for x in a]), a
"""


@functools.lru_cache(None)
def _lib() -> str:
    d = tempfile.mkdtemp(prefix="host_hip_")
    out = os.path.join(d, "libhosthip.so")
    cmd = ["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-w",
           "-I", os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include"),
           "-o", out, os.path.join(HERE, "host_hip.cpp")]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stdout + res.stderr
    return out


def run(source: str) -> str:
    prog = PRELUDE.format(root=ROOT, lib=_lib()) + textwrap.dedent(source)
    res = subprocess.run([sys.executable, "-c", prog], capture_output=True, text=True,
                         timeout=100)
    assert res.returncode == 0, res.stdout + res.stderr
    return res.stdout
