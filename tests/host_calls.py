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

    def batch(self, lps):
        """A block-diagonal batch of m x n LPs given as (m, n, counts)."""
        ms, ns, zs = ([f(l) for l in lps] for f in (lambda l: l[0], lambda l: l[1], lambda l: int(np.sum(l[2]))))
        off = [np.concatenate([[0], np.cumsum(v)]) for v in (ms, ns, zs)]
        rows, cols = [], []
        for (m, n, counts), r0, c0 in zip(lps, off[0], off[1]):
            rows += [r0 + np.sort((j + np.arange(k)) % m) for j, k in enumerate(counts)]
            cols += [np.full(k, c0 + j) for j, k in enumerate(counts)]
        rows, cols = np.concatenate(rows).astype(np.int32), np.concatenate(cols).astype(np.int32)
        order = np.lexsort((cols, rows))
        b = self.L.BatchStruct()
        b.count = len(lps)
        b.row_off, b.col_off = self.arr(off[0].astype(np.int32)), self.arr(off[1].astype(np.int32))
        b.nnz_off = self.arr(off[2].astype(np.int64))
        s = b.whole
        s.m, s.n, s.nnz = int(off[0][-1]), int(off[1][-1]), int(off[2][-1])
        s.a_rowptr = self.arr(np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=s.m))]).astype(np.int32))
        s.at_rowptr = self.arr(np.concatenate([[0], np.cumsum(np.bincount(cols, minlength=s.n))]).astype(np.int32))
        s.a_col, s.at_col = self.arr(cols[order]), self.arr(rows)
        s.a_val, s.at_val = self.arr(np.ones(rows.size)), self.arr(np.ones(rows.size))
        s.b, s.c = self.arr(np.ones(s.m)), self.arr(np.ones(s.n))
        return b

    def solve_batched(self, b, o, stream=0):
        nb = C.c_size_t(0)
        assert self.lib.mipdhg_batch_workspace_size(C.byref(b), C.byref(o), C.byref(nb)) == 0
        w = b.whole
        out = [self.buf(8 * k) for k in (w.n, w.m, w.n, w.m, w.n)]
        eps = self.arr(np.full(b.count, 1e-6))
        info = (self.L.InfoStruct * b.count)()
        return self.lib.mipdhg_solve_batched(C.byref(b), C.byref(o), eps, self.buf(nb.value), nb.value, stream, *out,
                                             info)

    def unrolled(self, b, o, stream=0, K=20, ckpt=10):
        nb = C.c_size_t(0)
        assert self.lib.mipdhg_unrolled_tape_size(C.byref(b), C.byref(o), K, ckpt, C.byref(nb)) == 0
        tape, w = self.buf(nb.value), b.whole
        rc = self.lib.mipdhg_unrolled_forward(C.byref(b), C.byref(o), K, ckpt, 0, tape, nb.value, stream,
                                              self.buf(8 * w.n))
        if rc < 0:
            return rc
        return self.lib.mipdhg_unrolled_backward(C.byref(b), C.byref(o), K, ckpt, tape, nb.value, self.buf(8 * w.n),
                                                 stream, self.buf(8 * w.n), self.buf(8 * w.m))

    def ipm(self, lp, ws, nbytes, stream=0, call="mipdhg_ipm_solve", start=True):
        o, info = self.L.IpmOptionsStruct(), self.L.IpmInfoStruct()
        self.lib.mipdhg_ipm_default_options(C.byref(o))
        out = [self.buf(8 * k) for k in (lp.n, lp.m, lp.n)]
        point = [self.arr(np.ones(k)) if start else None for k in (lp.n, lp.m, lp.n)]
        return getattr(self.lib, call)(C.byref(lp), None, None, *point, C.byref(o), ws, nbytes, stream, *out,
                                       C.byref(info))

    def errors_leave_nothing_running(self, call, names):
        """call() with each call of each of the runtime functions `names` made to fail once: it reports the error, and
        every stream that it launched a kernel on has been waited for since (a captured launch runs nothing).
        Returns the number of failures tried."""
        tried = 0
        for name in names:
            for skip in range(1000):
                self.shim.shim_reset()
                self.shim.shim_fail(name.encode(), skip)
                rc = call()
                log = self.log()
                if not any(w == "fail" for w, _, _ in log):
                    break
                tried += 1
                if rc >= 0:  # a failure that the call can do without
                    continue
                capturing, busy = set(), set()
                for w, n, s in log:
                    if w == "capture":
                        (capturing.add if n == "begin" else capturing.discard)(s)
                    elif (w == "kernel" and s not in capturing) or w == "graph":
                        busy.add(s)
                    elif w == "sync":
                        busy.discard(s)
                assert not busy, (name, skip, sorted(busy), log[-8:])
        return tried

    def log(self):
        """The calls since the last reset, as (what, name, stream)."""
        lines = [l.split(" ") for l in self.shim.shim_log().decode().splitlines()]
        return [(w, n, int(s, 16)) for w, n, s in lines]

    def kernels(self):
        return [n for w, n, _ in self.log() if w == "kernel"]
