"""Runs a piece of test code in a process of its own with hip_shim.c before the
HIP runtime: `shim` is that library, `mct2d`, `W`, `np` and `torch` are there,
and word(name) reads or sets one of its variables."""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))

PRELUDE = """
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
sys.path[:0] = [sys.argv[2], sys.argv[2] + "/tests"]
import numpy as np
import torch
from paper_2509_01827_amd import mct2d, workloads as W
from shimmed import CONFIGS, state
def word(name, value=None, type=ctypes.c_int):
    v = type.in_dll(shim, name)
    if value is not None:
        v.value = value
    return v.value
"""


def run(code, tmp_path, timeout=110):
    lib = str(tmp_path / "hip_shim.so")
    subprocess.check_call(["gcc", "-O1", "-fPIC", "-shared", "-o", lib, os.path.join(HERE, "hip_shim.c"), "-ldl"])
    r = subprocess.run([sys.executable, "-u", "-c", PRELUDE + code, lib, os.path.dirname(HERE)], timeout=timeout,
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    print(r.stdout, flush=True)
    assert r.returncode == 0


def CONFIGS():
    """Small models of every kind of resident step, cracks running."""
    from paper_2509_01827_amd import workloads as W
    grid = W.plate(45, 31, 0.0045, 0.0031, traction=2.0e7, jitter=0.02, seed=W.BASE_SEED + 45, notch_len=22, gc=0.0,
                   gc_field=W.weibull_gc(W.BASE_SEED + 31, 45 * 31, 6.0, 1.0), name="shimmed")
    return dict(grid=grid, grid32=dict(grid, precision=32), subcell=dict(grid, smoothing="subcell"),
                tri=W.tri_plate(40, 16, 0.1, 0.04, notch_len=0.05, traction=8.0e6),
                quad=W.quad_plate(24, 10, 0.1, 0.04, notch_len=0.05, traction=8.0e6))


def state(m):
    from paper_2509_01827_amd import mct2d
    lg = m.crack_set()
    return m.field(mct2d.FIELD_U) + m.field(mct2d.FIELD_V) + (m.split_codes(),) + tuple(lg[k] for k in sorted(lg))
