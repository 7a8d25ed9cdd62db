"""Runs test code on the library's host code without a GPU, in a process of its own: HIP is the
stand-in of fake_hip.cpp, torch a module of names (the binding's tensors are not used)."""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, sys, types
import numpy as np
sys.path.insert(0, {root!r})
hip = ctypes.CDLL({lib!r}, mode=ctypes.RTLD_GLOBAL)
for f in ("fake_live_count", "fake_live_bytes", "fake_mallocs", "fake_copies_from"):
    getattr(hip, f).restype = ctypes.c_longlong
hip.fake_fail_malloc_in.argtypes = [ctypes.c_longlong]
hip.fake_copies_from.argtypes = [ctypes.c_void_p]
torch = types.ModuleType("torch")
torch.autograd = types.SimpleNamespace(Function=object)
sys.modules["torch"] = torch
hip.fake_launches.restype = ctypes.c_char_p

def launches(known):  # which of these kernels ran since the last call, in order
    return [k for n in hip.fake_launches().decode().split() for k in known if str(len(k)) + k in n]
from paper_2402_08725_amd import starred as st
L = st.lib()
keep = []

def ptr(a):
    keep.append(a)
    return a.ctypes.data_as(ctypes.c_void_p)

def f32(n, v=0.0):
    return np.full(int(n), v, np.float32)

def make_plan(sides, ks, s, N, M, J, algo=st.CONV_FFT, mode=st.DECONV):
    sides, ks = np.array(sides, np.int32), np.array(ks, np.int32)
    d = st.Desc()
    d.mode, d.n_frames = mode, len(sides)
    d.side_host = sides.ctypes.data_as(ctypes.POINTER(ctypes.c_int32))
    d.ksize_host = ks.ctypes.data_as(ctypes.POINTER(ctypes.c_int32))
    d.subsample, d.grid_side, d.n_sources, d.n_scales = s, N, M, J
    d.w_pixel_stride, d.conv_algo, d.lambda_, d.gauss_fwhm = 0, algo, 1.0, 2.0
    h = ctypes.c_void_p()
    rc = L.starred_plan_create(ctypes.byref(d), None, ctypes.byref(h))
    assert rc == st.OK, (rc, L.starred_last_error())
    return h
"""


def run(tmp_path, code):
    """Python code run after PRELUDE; fails with its output if it does."""
    from paper_2402_08725_amd import build, starred
    if not os.path.exists(starred.LIB_PATH):
        build.build()
    lib = os.path.join(tmp_path, "libfake_hip.so")
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-o", lib, os.path.join(HERE, "fake_hip.cpp")], check=True)
    r = subprocess.run([sys.executable, "-c", PRELUDE.format(root=ROOT, lib=lib) + code], capture_output=True,
                       text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-4000:] + r.stderr[-4000:]
    return r.stdout
