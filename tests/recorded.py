"""The library with a recording HIP runtime (hip_record.cpp): its host code on the CPU, no kernel runs."""
import collections
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2010_09701_amd import build

Launch = collections.namedtuple("Launch", "kernel stream grid block lds nk")
Wait = collections.namedtuple("Wait", "stream event")
Record = collections.namedtuple("Record", "stream event")


def _library(d):
    objs = [os.path.join(build.ROOT, "_build", os.path.splitext(s)[0] + ".o") for s in build.SOURCES]
    if not all(map(os.path.exists, objs)):
        pytest.skip("objects of the library are not there (run __graft_entry__.build())")
    lib, stub = os.path.join(d, "liboefe_rec.so"), os.path.join(os.path.dirname(os.path.abspath(__file__)), "hip_record.cpp")
    # the test runtime's own definitions, whatever else the process has loaded
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-Wno-attributes",
                    "-I" + os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include"), stub, *objs,
                    "-Wl,-Bsymbolic", "-o", lib], check=True, capture_output=True)
    return ctypes.CDLL(lib)


class Recorded:
    def __init__(self, d):
        """d: a directory for the library"""
        from paper_2010_09701_amd import oefe
        self.desc = oefe._Desc
        self.lib = _library(d)
        self.lib.rec_log.restype = ctypes.c_char_p
        for f in ("oefe_work_size", "oefe_batched_work_size"):
            getattr(self.lib, f).restype = ctypes.c_size_t
        self.lib.oefe_last_error.restype = ctypes.c_char_p
        self._keep = []

    def operator(self, s, poisson=False):
        atom, power, zeta, axis = s.enr_arrays()
        k = [np.ascontiguousarray(s.pos, dtype=np.float64).ravel(), np.ascontiguousarray(s.Z, dtype=np.float64), atom,
             power, zeta, axis, None if s.kvec is None else np.ascontiguousarray(s.kvec, dtype=np.float64)]
        self._keep.append(k)
        P = lambda a, t: None if a is None else a.ctypes.data_as(ctypes.POINTER(t))
        dbl, i32 = ctypes.c_double, ctypes.c_int32
        d = self.desc(s.L, s.nc, s.p, s.n_atoms, P(k[0], dbl), P(k[1], dbl), s.sigma, s.r0, s.r1, s.n_enr, P(atom, i32),
                      P(power, i32), P(zeta, dbl), P(axis, i32), P(k[6], dbl))
        h = ctypes.c_void_p(0)
        rc = (self.lib.oefe_poisson_create if poisson else self.lib.oefe_op_create)(ctypes.byref(d), ctypes.byref(h))
        assert rc == 0, self.lib.oefe_last_error()
        return h

    def events(self):
        """What was queued since the last call, in order."""
        out = []
        for ln in self.lib.rec_log().decode().splitlines():
            w = ln.split()
            if w[0] == "launch":
                out.append(Launch(w[1], *map(int, w[2:])))
            else:
                out.append((Wait if w[0] == "wait" else Record)(*map(int, w[1:])))
        self.lib.rec_clear()
        return out

    def fail_attribute(self, part=""):
        self.lib.rec_fail_attribute(part.encode())

    def filter(self, h, prec, n_tot, nv, m, stream=7):
        """chebyshev_filter of a block of ones on stream `stream`; returns its status."""
        x = np.ones((n_tot, nv, 2))
        work = np.zeros(int(self.lib.oefe_work_size(h, prec, nv)) + 256, dtype=np.uint8)
        dbl = ctypes.c_double
        return self.lib.chebyshev_filter(h, prec, x.ctypes.data_as(ctypes.c_void_p), ctypes.c_int64(nv), nv, m, dbl(1.0),
                                         dbl(2.0), dbl(0.0), work.ctypes.data_as(ctypes.c_void_p), ctypes.c_void_p(stream))

    def batched(self, hs, prec, n_tot, nv, m, stream=7):
        nk = len(hs)
        xs = [np.ones((n_tot, nv, 2)) for _ in hs]
        H = (ctypes.c_void_p * nk)(*[h.value for h in hs])
        X = (ctypes.c_void_p * nk)(*[x.ctypes.data for x in xs])
        LD, NV = (ctypes.c_int64 * nk)(*[nv] * nk), (ctypes.c_int32 * nk)(*[nv] * nk)
        abc = (ctypes.c_double * (3 * nk))(*[1.0, 2.0, 0.0] * nk)
        work = np.zeros(int(self.lib.oefe_batched_work_size(nk, H, prec, NV)) + 256, dtype=np.uint8)
        return self.lib.chebyshev_filter_batched(nk, H, prec, X, LD, NV, m, abc, work.ctypes.data_as(ctypes.c_void_p),
                                                 ctypes.c_void_p(stream))

    def autotune(self, hs, prec, n_tot, nv, reps=2, stream=7):
        """(status, cw, cb)"""
        nk = len(hs)
        xs = [np.ones((n_tot, nv, 2)) for _ in hs]
        H = (ctypes.c_void_p * nk)(*[h.value for h in hs])
        X = (ctypes.c_void_p * nk)(*[x.ctypes.data for x in xs])
        LD, NV = (ctypes.c_int64 * nk)(*[nv] * nk), (ctypes.c_int32 * nk)(*[nv] * nk)
        work = np.zeros(int(self.lib.oefe_batched_work_size(nk, H, prec, NV)) + 256, dtype=np.uint8)
        cw, cb, ms = ctypes.c_int32(-1), ctypes.c_int32(-1), ctypes.c_double(0)
        rc = self.lib.oefe_autotune(nk, H, prec, X, LD, NV, reps, work.ctypes.data_as(ctypes.c_void_p), ctypes.byref(cw),
                                    ctypes.byref(cb), ctypes.byref(ms), ctypes.c_void_p(stream))
        return rc, cw.value, cb.value

    def apply(self, h, prec, n_tot, nv, stream=7):
        x, y = np.ones((n_tot, nv, 2)), np.ones((n_tot, nv, 2))
        work = np.zeros(int(self.lib.oefe_work_size(h, prec, nv)) + 256, dtype=np.uint8)
        p = [a.ctypes.data_as(ctypes.c_void_p) for a in (x, y, work)]
        return self.lib.ham_apply(h, prec, p[0], p[1], ctypes.c_int64(nv), nv, p[2], ctypes.c_void_p(stream))
