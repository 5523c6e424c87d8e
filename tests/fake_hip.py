"""The library on a HIP runtime without a device (fake_hip.cpp), for CPU tests of
its host code.  Run as a program: `python fake_hip.py <fake runtime> <scenario
module> <scenario>` calls the scenario with a Fake."""
import ctypes as C
import importlib
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.dirname(os.path.abspath(__file__))


def build(out_dir) -> str:
    so = os.path.join(str(out_dir), "libfakehip.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-w",
                           "-I/opt/rocm/include", os.path.join(HERE, "fake_hip.cpp"), "-o", so])
    return so


def run(so, module, scenario):
    """The scenario in a process of its own (the fake runtime stays out of the tests' one)."""
    r = subprocess.run([sys.executable, os.path.abspath(__file__), so, module, scenario], capture_output=True, text=True,
                       cwd=ROOT, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr


class Fake:
    """The fake runtime's controls and the library's functions."""

    def __init__(self, so):
        self.rt = C.CDLL(so, mode=C.RTLD_GLOBAL)
        self.rt.fake_memory.argtypes = [C.c_size_t]
        self.rt.fake_used.restype = C.c_size_t
        self.rt.fake_launch.restype = C.c_char_p
        self.rt.fake_launch.argtypes = [C.c_int, C.POINTER(C.c_uint64)]
        import paper_2506_20043_amd as pv
        self.pv, self.lib = pv, pv.lib()

    def context(self, device=0):
        """What the binding's classes need of a Context (which would import torch)."""
        h = C.c_void_p()
        assert self.lib.pv_create(device, C.byref(h)) == 0
        return type("Ctx", (), {"h": h, "device": device})()

    def grids(self, ctx, n_atoms=50, boxes=(([5., 5, 5], 10., 0.5),)):
        import numpy as np
        pv = self.pv
        g = np.random.default_rng(1)
        x, t = g.random((n_atoms, 3), dtype=np.float32) * 10, g.integers(0, 8, n_atoms).astype(np.uint8)
        b, h = pv.make_boxes(list(boxes)), C.c_void_p()
        st = self.lib.pv_build_grids(ctx.h, n_atoms, x.ctypes.data, t.ctypes.data, b, len(b), 10.0, None, C.byref(h))
        return pv.Grids(ctx, h, len(b)) if st == 0 else st

    def launches(self, name=""):
        """(name, grid, block, LDS, stream) of the launches since the last call whose kernel's name holds `name`."""
        out = []
        for i in range(self.rt.fake_launches()):
            v = (C.c_uint64 * 8)()
            k = self.rt.fake_launch(i, v).decode()
            if name in k:
                out.append((k, tuple(v[0:3]), tuple(v[3:6]), v[6], v[7]))
        self.rt.fake_clear()
        return out


if __name__ == "__main__":
    sys.path[:0] = [ROOT, HERE]
    getattr(importlib.import_module(sys.argv[2]), sys.argv[3])(Fake(sys.argv[1]))
