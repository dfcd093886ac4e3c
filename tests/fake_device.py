"""Calls into libfwime.so on the device-less HIP runtime of fake_hip.cpp.

Run as a script, in a process of its own: `python fake_device.py FAKE_SO CODE`
executes CODE with `Fake` in scope and without importing torch (whose own HIP
libraries would bind to the stand-in).  Device addresses are dummies.
"""
import ctypes
import importlib.util
import os
import sys
import types

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PTR = 1 << 45                                   # stands for any caller's device array
GiB = 1 << 30


class Fake:
    """One context on a device of `size` bytes of which others hold `other`."""

    def __init__(self, size=288 * GiB, other=0, budget=0):
        self.hip.fake_device(size, other)
        self.hip.fake_largest(2 ** 64 - 1)
        h = ctypes.c_void_p()
        assert self.lib.fwime_ctx_create(0, budget, ctypes.byref(h)) == 0
        self.h, self.keep = h, []

    def problem(self, nz, nx, nt, shots, nb=40, rec=None):
        rec = np.arange(nx) if rec is None else rec
        iz = [np.zeros(shots, np.int32), np.zeros(shots, np.int32), np.zeros((shots, len(rec)), np.int32),
              np.ascontiguousarray(np.tile(rec, (shots, 1)), np.int32)]
        self.keep.append(iz)
        g = self.abi._Grid(nz, nx, nb, nt, 10.0, 10.0, 8e-4, 0.3, 0)
        geo = self.abi._Geom(shots, len(rec), *(a.ctypes.data for a in iz), PTR)
        return ctypes.byref(g), ctypes.byref(geo), g, geo

    def model(self, p):
        return self.lib.fwime_model(self.h, p[0], PTR, p[1], PTR, None)

    def born_fwd(self, p, nh):
        return self.lib.fwime_born_ext_fwd(self.h, p[0], PTR, p[1], nh, PTR, PTR, None)

    def born_adj(self, p, nh):
        return self.lib.fwime_born_ext_adj(self.h, p[0], PTR, p[1], nh, PTR, PTR, None)

    def gradient(self, p, nh):
        dso = np.ones(nh)
        return self.lib.fwime_gradient(self.h, p[0], PTR, p[1], nh, PTR, PTR, 1e-3, dso.ctypes.data, PTR, PTR, PTR, None)

    def vp(self, p, nh, niter=1):
        dso, phi = np.ones(nh), np.zeros(niter + 1)
        return self.lib.fwime_vp_solve(self.h, p[0], PTR, p[1], nh, PTR, 1e-3, dso.ctypes.data, niter, PTR,
                                       phi.ctypes.data, None)

    def spline(self, nz, nx, zn, xn, adjoint):
        zn, xn = (np.ascontiguousarray(a, np.float64) for a in (zn, xn))
        f = self.lib.fwime_spline_adjoint if adjoint else self.lib.fwime_spline_apply
        return f(self.h, nz, nx, 10.0, 10.0, len(zn), zn.ctypes.data, len(xn), xn.ctypes.data, PTR, PTR, None)

    def lbfgs(self, n, pairs):
        return self.lib.fwime_lbfgs_direction(self.h, n, pairs, PTR, PTR, PTR, PTR, None)

    def engine(self, max_jobs):
        e = ctypes.c_void_p()
        rc = self.lib.fwime_engine_create(self.h, 64, max_jobs, None, ctypes.byref(e))
        return rc, e

    def submit(self, engine, p):
        job, ticket = self.abi._Job(p[2], PTR, p[3], PTR), ctypes.c_int64()
        return self.lib.fwime_engine_submit(engine, ctypes.byref(job), None, ctypes.byref(ticket))

    def forward(self, p, nh):
        t = ctypes.c_void_p()
        rc = self.lib.fwime_forward_tape(self.h, p[0], PTR, p[1], nh, PTR, PTR, ctypes.byref(t), None)
        return rc, t

    def backward(self, tape):
        return self.lib.fwime_backward_tape(self.h, tape, PTR, PTR, PTR, None)

    def free(self, tape):
        self.lib.fwime_tape_free(tape)

    def trim(self):
        assert self.lib.fwime_ctx_trim(self.h, None) == 0

    def info(self):
        out = self.abi._Info()
        assert self.lib.fwime_ctx_info(self.h, ctypes.byref(out)) == 0
        return out

    def held(self):
        n = ctypes.c_size_t()
        assert self.lib.fwime_ctx_held(self.h, ctypes.byref(n)) == 0
        return n.value

    def error(self):
        return self.lib.fwime_last_error(self.h).decode()

    def close(self):
        self.lib.fwime_ctx_destroy(self.h)

    @property
    def used(self):
        return self.hip.fake_used()

    @property
    def peak(self):
        return self.hip.fake_peak()

    @property
    def allocations(self):
        return self.hip.fake_allocations()

    def footprint(self, p, nrec, nh, op):
        n = ctypes.c_size_t()
        assert self.lib.fwime_footprint(p[0], p[3].nshots, nrec, nh, op, ctypes.byref(n)) == 0
        return n.value

    def launched(self, part):
        return self.hip.fake_launched(part.encode())


def _load(fake_so):
    hip = ctypes.CDLL(fake_so, mode=ctypes.RTLD_GLOBAL)
    for f in ("fake_used", "fake_peak"):
        getattr(hip, f).restype = ctypes.c_size_t
    hip.fake_allocations.restype = ctypes.c_long
    hip.fake_device.argtypes = [ctypes.c_size_t, ctypes.c_size_t]
    hip.fake_largest.argtypes = [ctypes.c_size_t]
    hip.fake_launched.argtypes, hip.fake_launched.restype = [ctypes.c_char_p], ctypes.c_long
    sys.modules["torch"] = types.ModuleType("torch")
    spec = importlib.util.spec_from_file_location("_abi", os.path.join(ROOT, "paper_2206_02362_amd", "_abi.py"))
    abi = sys.modules["_abi"] = importlib.util.module_from_spec(spec)
    sys.modules["torch"].Tensor = type("Tensor", (), {})
    spec.loader.exec_module(abi)
    Fake.hip, Fake.abi, Fake.lib = hip, abi, abi.load()


if __name__ == "__main__":
    _load(sys.argv[1])
    exec(sys.argv[2], {"Fake": Fake, "GiB": GiB, "PTR": PTR, "ctypes": ctypes, "np": np})
