"""Runs the host code of libmipdhg.so against the stand-in HIP runtime of
hip_host_calls.c: which kernels a call launches, on which streams, and what it
has waited for when it returns.  No GPU, no torch; a process of its own, whose
HIP symbols are the stand-in's (test_host_calls.py starts it)."""
import ctypes as C
import importlib.util
import os
import sys
import types

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


class Host:
    def __init__(self, shim):
        self.shim = C.CDLL(shim, mode=C.RTLD_GLOBAL)
        self.shim.shim_log.restype = C.c_char_p
        sys.modules["torch"] = types.ModuleType("torch")  # the bindings' structs only
        spec = importlib.util.spec_from_file_location("_lib", os.path.join(ROOT, "paper_2603_03150_amd", "_lib.py"))
        self.L = importlib.util.module_from_spec(spec)
        spec.loader.exec_module(self.L)
        self.lib = C.CDLL(self.L.LIB_PATH)
        for name, (res, args) in self.L.SIGNATURES.items():
            f = getattr(self.lib, name)
            f.restype, f.argtypes = res, args
        self.keep = []

    def options(self, precision="fp64", **kw):
        o = self.L.OptionsStruct()
        self.lib.mipdhg_default_options(C.byref(o))
        o.precision = self.L.PRECISION[precision]
        for k, v in kw.items():
            setattr(o, k, v)
        return o

    def buf(self, nbytes, align=256):
        a = np.zeros(nbytes + align, dtype=np.uint8)
        self.keep.append(a)
        return (a.ctypes.data + align - 1) // align * align

    def arr(self, a):
        a = np.ascontiguousarray(a)
        self.keep.append(a)
        return a.ctypes.data

    def lp(self, m, n, counts):
        """counts[j] entries in column j, rows j, j + 1, ... modulo m."""
        rows = np.concatenate([np.sort((j + np.arange(k)) % m) for j, k in enumerate(counts)] or [[]]).astype(np.int32)
        cols = np.repeat(np.arange(n), counts).astype(np.int32)
        order = np.lexsort((cols, rows))
        s = self.L.LPStruct()
        s.m, s.n, s.nnz = m, n, rows.size
        s.a_rowptr = self.arr(np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=m))]).astype(np.int32))
        s.at_rowptr = self.arr(np.concatenate([[0], np.cumsum(counts)]).astype(np.int32))
        s.a_col, s.at_col = self.arr(cols[order]), self.arr(rows)
        s.a_val = self.arr(np.ones(rows.size))
        s.at_val = self.arr(np.ones(rows.size))
        s.b, s.c = self.arr(np.ones(m)), self.arr(np.ones(n))
        return s

    def solve(self, lp, o, stream=0):
        nb = C.c_size_t(0)
        assert self.lib.mipdhg_workspace_size(C.byref(lp), C.byref(o), C.byref(nb)) == 0
        out = [self.buf(8 * k) for k in (lp.n, lp.m, lp.n, lp.m, lp.n, lp.m, lp.n)]
        ws = self.buf(nb.value)
        info = self.L.InfoStruct()
        return self.lib.mipdhg_solve(C.byref(lp), C.byref(o), 1e-6, ws, nb.value, stream, *out, C.byref(info))

    def log(self):
        """The calls since the last reset, as (what, name, stream)."""
        lines = [l.split(" ") for l in self.shim.shim_log().decode().splitlines()]
        return [(w, n, int(s, 16)) for w, n, s in lines]

    def kernels(self):
        return [n for w, n, _ in self.log() if w == "kernel"]
