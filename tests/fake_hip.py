"""Runs the library's host code on a HIP runtime without a device
(fake_hip.cpp), in a process of its own."""
import ctypes
import os
import shutil
import subprocess
import sys

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def build(folder):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    so = str(folder / "libfakehip.so")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-pthread",
                        os.path.join(HERE, "fake_hip.cpp"), "-o", so], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return so


def run(folder, code):
    """The Python `code` with `hip` (set, notes) and `context` (below) at hand; its output."""
    head = f"import sys; sys.path[:0] = [{ROOT!r}, {HERE!r}]\nimport fake_hip\nhip = fake_hip.load({build(folder)!r})\n" \
           "from fake_hip import context, call, abi\n"
    r = subprocess.run([sys.executable, "-c", head + code], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout


class load:
    def __init__(self, so):
        self.so = ctypes.CDLL(so, mode=ctypes.RTLD_GLOBAL)
        self.so.fake_hip_notes.restype = ctypes.c_char_p

    def set(self, pinned_fails=0, in_capture=0):
        self.so.fake_hip_set(pinned_fails, in_capture)

    def notes(self):
        return self.so.fake_hip_notes().decode().splitlines()


if ROOT not in sys.path:
    sys.path.insert(0, ROOT)
from paper_1611_02445_amd import _abi as abi  # noqa: E402
from paper_1611_02445_amd._abi import call  # noqa: E402


class context:
    """A context over host memory that stands for the device's (as much of it as a call touches)."""

    def __init__(self, solid, periodic=7, **params):
        solid = np.ascontiguousarray(solid, dtype=np.uint8)
        self.tiles = ctypes.POINTER(abi.Tiles)()
        nz, ny, nx = solid.shape
        call("lbm_build_tiles", solid.ctypes.data_as(ctypes.c_void_p), nx, ny, nz, periodic, ctypes.byref(self.tiles))
        p = abi.Params(tau=0.7, rho0=1.0, **params)
        size = abi.Sizes()
        call("lbm_required_bytes", self.tiles, ctypes.byref(p), ctypes.byref(size))
        self.size = size
        self.buffers = [np.zeros(n + 256, np.uint8) for n in (size.table_bytes, size.scratch_bytes)]
        table, scratch = (ctypes.c_void_p((b.ctypes.data + 255) // 256 * 256) for b in self.buffers)
        # the lattices are addresses that nothing reads
        self.state = [ctypes.c_void_p(1 << 40), ctypes.c_void_p(1 << 41)]
        self.ctx = ctypes.c_void_p()
        call("lbm_create", self.tiles, ctypes.byref(p), *self.state, table, scratch, None, ctypes.byref(self.ctx))

    def sums(self):
        s = (ctypes.c_double * 8)()
        call("lbm_macroscopic", self.ctx, None, None, s)
        return list(s)

    def destroy(self):
        call("lbm_destroy", self.ctx)
        self.ctx = None
