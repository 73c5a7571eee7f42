"""Windows on cache lines: of a large filter's windows of 1024 weights, whose
places are uniform over all of them, nearly all begin on a 128-byte line whatever
the filter's size, so that a wave reads two lines per step; and every window
lies inside the memory set aside. (CPU: the records' layout, from the library's
own header.)"""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "helpers", "filter_windows.cpp")
CSRC = os.path.join(os.path.dirname(HERE), "paper_2109_13504_amd", "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
W, AUX, TILE = 1 << 40, 1 << 41, 1024  # addresses, a multiple of any line; particles per block at most


@pytest.fixture(scope="module")
def layout(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("needs hipcc")
    out = str(tmp_path_factory.mktemp("windows") / "filter_windows.so")
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-fPIC", "-shared", "-I", INCLUDE,
                    "-I", CSRC, "-o", out, SRC], check=True, cwd="/tmp")
    lib = ctypes.CDLL(out)
    lib.filter_windows.argtypes = [ctypes.c_uint64, ctypes.c_uint64, ctypes.c_uint32, ctypes.c_uint32, ctypes.c_int,
                                   ctypes.POINTER(ctypes.c_uint64)]
    lib.filter_windows.restype = None

    def f(n, B, in_place):
        o = (ctypes.c_uint64 * 4)()
        lib.filter_windows(W, AUX, n, B, in_place, o)
        return list(o)

    return f


@pytest.mark.parametrize("in_place", [1, 0])
@pytest.mark.parametrize("n,B", [(1000, 60), (1 << 20, 354), ((1 << 20) + 32, 0), (1 << 24, 354), ((1 << 22) + 13, 300),
                                 (6000001, 354), (15000001, 354), (15000001, 0), ((1 << 24) - 5, 100),
                                 ((1 << 29) - 4096 - 1, 60), ((1 << 29) - 4096, 60)])
def test_windows(layout, n, B, in_place):
    w, past, runs_on, floats = layout(n, B, in_place)
    g = np.random.default_rng(n % 1000)
    start = g.integers(0, (n + TILE - 1) // TILE, 40000) * TILE
    s = start + g.integers(0, n, start.size) // 32 * 32
    if not runs_on:
        s = np.where(s >= n, s - n, s)
    inside = s + TILE <= n
    at = np.where(inside, w, past).astype(np.uint64) + (4 * s).astype(np.uint64)
    assert (4 * s + 4 * TILE < 1 << 32).all()  # byte offsets are 32 bits
    if n > 1 << 20:
        assert (at % 128 == 0).mean() > 0.99
    if in_place:
        assert (at[inside] >= W).all() and (at[inside] + 4 * TILE <= W + 4 * n).all()
    aux = at if not in_place else at[~inside]
    assert (aux >= AUX).all() and (aux + 4 * TILE <= AUX + 4 * floats).all()
