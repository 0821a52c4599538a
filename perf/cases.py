"""The work this library is measured on: PDHG solves of one LP, batches of LPs, the differentiable unrolled map, and
the interior-point hybrid, each through the entry points of paper_2603_03150_amd.

All LPs are synthetic with a planted optimum (b = A x*, c = A^T y* + z*, x* and z* complementary), drawn on the GPU
from the case's seed; the recipes (uniform columns, power-law columns with row factors, diagonal blocks with linking
rows, the general form's mix of bounds and senses) are those of lpgen.  Solves are cut at an iteration limit, so that
the work of a pass is known: the iterations, evaluations and restarts are those of a longer solve.

FP32 and BF16 solves hold their iterates in float32, and their point (x, y, z), what the interior-point method is
handed, is returned in that type; their residual vectors are the float64 differences that the rounding of that point
leaves, so they are returned where the point is float64, from the FP64 solves.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2603_03150_amd as P

DEV = "cuda"
F64 = torch.float64
EVAL_EVERY = 64      # the library's defaults
POWER_ITERS = 100
RUIZ = 10
VALUE_BYTES = {"fp64": 8, "fp32": 4, "bf16": 2}
STATE_BYTES = {"fp64": 8, "fp32": 4, "bf16": 4}


# ---------------------------------------------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------------------------------------------
def listed() -> list[dict]:
    return [
        # The smallest solve: the 200 x 500 LP of the tests and the smoke run, where launches and host work count.
        dict(name="solve_small_fp64", kind="solve", lp="uniform", m=200, n=500, per_col=5, precision="fp64", iters=256),
        # An ordinary solve of ragged size whose matrix is kept in BF16.
        dict(name="solve_power_law_bf16", kind="solve", lp="power_law", m=25013, n=99991, precision="bf16", iters=256),
        # The benchmark's power-law LP in the usual FP32 mode, with the default kernel shapes.
        dict(name="solve_power_law_fp32", kind="solve", lp="power_law", m=100000, n=400000, precision="fp32",
             iters=512),
        # The general form (bounds, inequality rows) at an odd size.
        dict(name="solve_general_fp32", kind="solve", lp="general", m=50021, n=200003, precision="fp32", iters=256),
        # The benchmark's block-angular LP, the largest single LP, with the kernel shapes its autotuner picks: the
        # only one that does not fit the last-level cache.
        dict(name="solve_block_angular_fp32", kind="solve", lp="block", nblocks=64, bm=30000, bn=120000, nlink=2000,
             link_nnz=1200, precision="fp32", iters=256),
        # The benchmark's batch: 4,096 LPs of very uneven size.
        dict(name="batch_4096_fp32", kind="batch", count=4096, m_lo=20, m_hi=2000, precision="fp32", iters=256),
        # A small batch in the parity precision: fewer instances than compute units.
        dict(name="batch_48_fp64", kind="batch", count=48, m_lo=20, m_hi=500, precision="fp64", iters=256),
        # The benchmark's differentiation workload (a training step: x_K, dL/dc, dL/db) at a shorter K.
        dict(name="unrolled_256_fp32", kind="unrolled", count=256, m=500, n=1500, per_col=5, precision="fp32", K=400,
             ckpt=100),
        # The finite-difference set of the tests: tiny instances, latency only.
        dict(name="unrolled_16_fp64", kind="unrolled", count=16, m=20, n=50, per_col=5, precision="fp64", K=200,
             ckpt=100),
        # The interior-point consumer from a cold start on the middle size of the hybrid benchmark.
        dict(name="ipm_cold_1000", kind="ipm_cold", lp="power_law", m=1000, n=4000, steps=6),
        # The same at its largest size: dense factorisations of order 4,000.
        dict(name="ipm_cold_4000", kind="ipm_cold", lp="power_law", m=4000, n=16000, steps=3),
        # The hybrid's warm start (Algorithm 1 and the Newton step that decides whether the start is kept) on its
        # smallest size.
        dict(name="ipm_warm_200", kind="ipm_warm", lp="uniform", m=200, n=500, per_col=5, steps=1),
    ]


def _log(rng, lo, hi) -> int:
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng) -> dict:
    kind = rng.choices(["solve", "general", "block", "batch", "unrolled", "ipm_cold", "ipm_warm"],
                       [5, 2, 2, 4, 3, 2, 2])[0]
    if kind in ("solve", "general"):
        m = _log(rng, 200, 100000)
        case = dict(kind="solve", lp="general", m=m, n=int(m * rng.uniform(2.0, 4.0)),
                    precision=rng.choice(["fp64", "fp32", "fp32", "bf16"]), iters=rng.choice([128, 192, 256]))
        if kind == "solve":
            case["lp"] = rng.choice(["uniform", "power_law"])
            if case["lp"] == "uniform":
                case["per_col"] = rng.randint(3, 12)
        return case
    if kind == "block":
        bm = _log(rng, 1000, 30000)
        return dict(kind="solve", lp="block", nblocks=rng.randint(4, 48), bm=bm, bn=4 * bm, nlink=rng.randint(50, 2000),
                    link_nnz=rng.randint(100, 1200), precision=rng.choice(["fp32", "fp32", "bf16"]),
                    iters=rng.choice([128, 256]))
    if kind == "batch":
        lo = _log(rng, 20, 200)
        return dict(kind="batch", count=_log(rng, 8, 4000), m_lo=lo, m_hi=lo * rng.randint(1, 10),
                    precision=rng.choice(["fp64", "fp32", "fp32", "bf16"]), iters=rng.choice([128, 256]))
    if kind == "unrolled":
        m = _log(rng, 20, 500)
        return dict(kind="unrolled", count=_log(rng, 4, 256), m=m, n=int(m * rng.uniform(2.0, 3.0)),
                    per_col=rng.randint(3, 6), precision=rng.choice(["fp32", "fp64"]), K=rng.randint(100, 400),
                    ckpt=rng.choice([50, 100]))
    if kind == "ipm_cold":
        m = _log(rng, 200, 3000)
        return dict(kind="ipm_cold", lp="power_law", m=m, n=int(m * rng.uniform(3.0, 4.0)), steps=rng.randint(2, 6))
    m = _log(rng, 100, 2000)
    return dict(kind="ipm_warm", lp="uniform", m=m, n=int(m * rng.uniform(2.0, 3.0)), per_col=rng.randint(4, 6),
                steps=1)


# ---------------------------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------------------------
class _Csr:
    """A CSR matrix as DeviceLP reads it."""

    def __init__(self, shape, row, col, val):
        self.shape = shape
        self.nnz = int(col.numel())
        ptr = torch.zeros(shape[0] + 1, dtype=torch.int64, device=row.device)
        ptr[1:] = torch.bincount(row, minlength=shape[0]).cumsum(0)
        self.indptr = ptr.to(torch.int32).cpu().numpy()
        self.indices = col.to(torch.int32).cpu().numpy()
        self.data = val.cpu().numpy()


def _gen(seed: int) -> torch.Generator:
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _u(g, n, lo=0.0, hi=1.0):
    return torch.rand(n, generator=g, device=DEV, dtype=F64) * (hi - lo) + lo


def _uniform_rows(g, n, k, base, span):
    """k distinct rows for each of n columns, in [base, base + span) (per-column tensors or numbers)."""
    base = torch.as_tensor(base, device=DEV).expand(n)[:, None]
    span = torch.as_tensor(span, device=DEV).expand(n)[:, None].to(F64)

    def pick(shape):
        return torch.rand(shape, generator=g, device=DEV, dtype=F64)

    rows = torch.minimum((pick((n, k)) * span).long(), span.long() - 1)
    while True:
        rows = rows.sort(dim=1).values
        dup = torch.zeros_like(rows, dtype=torch.bool)
        dup[:, 1:] = rows[:, 1:] == rows[:, :-1]
        if not bool(dup.any()):
            return rows + base
        again = torch.minimum((pick((n, k)) * span).long(), span.long() - 1)
        rows = torch.where(dup, again, rows)


def _pattern(case, g):
    """(m, n, row, col, values) of a single LP's matrix, column-major with increasing rows."""
    lp = case["lp"]
    if lp == "block":
        nb, bm, bn = case["nblocks"], case["bm"], case["bn"]
        m, n = nb * bm + case["nlink"], nb * bn
        cols = torch.arange(n, device=DEV)
        rows = _uniform_rows(g, n, 6, (cols // bn) * bm, bm)
        lcol = (torch.rand((case["nlink"], case["link_nnz"]), generator=g, device=DEV, dtype=F64) * n).long()
        lrow = torch.arange(case["nlink"], device=DEV)[:, None].expand_as(lcol) + nb * bm
        key = torch.cat([(cols[:, None] * m + rows).reshape(-1), (lcol * m + lrow).reshape(-1)])
    elif lp == "uniform":
        m, n, k = case["m"], case["n"], min(case["per_col"], case["m"])
        rows = _uniform_rows(g, n, k, 0, m)
        key = (torch.arange(n, device=DEV)[:, None] * m + rows).reshape(-1)
    else:  # power-law column counts, 2 to 2,000 with mean 8
        m, n = case["m"], case["n"]
        k = torch.arange(2, min(2000, m) + 1, device=DEV, dtype=F64)
        cdf = (k ** -2.1423).cumsum(0)
        counts = (torch.searchsorted(cdf / cdf[-1], _u(g, n)).clamp(max=k.numel() - 1) + 2).long()
        col = torch.repeat_interleave(torch.arange(n, device=DEV), counts)
        key = col * m + (_u(g, col.numel()) * m).long().clamp(max=m - 1)
    key = torch.unique(key)  # sorted; a column's repeated rows fall together
    col = key // m
    row = key - col * m
    val = torch.randn(key.numel(), generator=g, device=DEV, dtype=F64)
    if lp in ("power_law", "general"):
        val = val * _u(g, m, 0.1, 10.0)[row]
    return m, n, row, col, val


def _by_row(row, v, m, reduce="sum"):
    """v summed (or its maximum taken) over each of m rows; row is sorted."""
    return torch.segment_reduce(v, reduce, lengths=torch.bincount(row, minlength=m), initial=0)


def _mul(row, col, val, x, m):
    return _by_row(row, val * x[col], m)


def _problem(case, seed) -> dict:
    """The LP (or the block-diagonal LP of a batch) as device tensors in float64."""
    g = _gen(seed)
    p = dict(lo=None, hi=None, sense=None)
    if case["kind"] in ("batch", "unrolled"):
        ms, ns = _sizes(case)
        ro = torch.as_tensor(np.concatenate([[0], np.cumsum(ms)]), device=DEV)
        co = torch.as_tensor(np.concatenate([[0], np.cumsum(ns)]), device=DEV)
        ci = torch.repeat_interleave(torch.arange(len(ns), device=DEV), torch.as_tensor(ns, device=DEV))
        m, n, k = int(ro[-1]), int(co[-1]), case.get("per_col", 4)
        rows = _uniform_rows(g, n, k, ro[ci], torch.as_tensor(ms, device=DEV)[ci])
        row, col = rows.reshape(-1), torch.arange(n, device=DEV)[:, None].expand(n, k).reshape(-1)
        val = torch.randn(row.numel(), generator=g, device=DEV, dtype=F64)
        p.update(row_off=ro, col_off=co)
    else:
        m, n, row, col, val = _pattern(case, g)
    order = torch.argsort(row * n + col)
    on = torch.rand(n, generator=g, device=DEV) < 0.5
    x = torch.where(on, _u(g, n), 0.0)
    y = torch.randn(m, generator=g, device=DEV, dtype=F64)
    z = torch.where(on, 0.0, _u(g, n))
    b0 = torch.zeros(m, device=DEV, dtype=F64)
    if case.get("lp") == "general":
        # 30 % [0, inf), 25 % boxes, 10 % free, 15 % (-inf, u], 20 % [l, inf); half the rows =, a quarter >=, <= each
        kind = torch.bucketize(_u(g, n), torch.tensor([0.3, 0.55, 0.65, 0.8], device=DEV, dtype=F64))
        inf = math.inf
        l1, wd, ub = _u(g, n, -1.0, 0.0), _u(g, n, 0.5, 2.0), _u(g, n, -1.0, 1.0)
        lo = torch.where(kind == 0, 0.0, torch.where(kind == 1, l1, torch.where(kind == 4, ub, -inf)))
        hi = torch.where(kind == 1, l1 + wd, torch.where(kind == 3, ub, inf))
        u, t, lam = _u(g, n), _u(g, n), _u(g, n)
        at_hi = (kind == 3) & (u < 0.5) | (kind == 1) & (u < 1 / 3)
        at_lo = ((kind == 0) | (kind == 4)) & (u < 0.5) | (kind == 1) & (u > 2 / 3)
        x = torch.where(kind == 1, lo + t * wd, torch.where(kind == 3, hi - t, torch.where(kind == 2, y.new_tensor(2.0) * t - 1.0, lo + t)))
        x = torch.where(at_lo, lo, torch.where(at_hi, hi, x))
        z = torch.where(at_lo, lam, torch.where(at_hi, -lam, 0.0))
        sense = torch.bucketize(_u(g, m), torch.tensor([0.5, 0.75], device=DEV, dtype=F64))
        active = _u(g, m) < 0.6
        y = torch.where(sense == 0, y, torch.where(active, torch.where(sense == 1, y.abs(), -y.abs()), 0.0))
        slack = torch.where((sense != 0) & ~active, _u(g, m, 0.1, 1.0), 0.0)
        b0 = torch.where(sense == 1, -slack, slack)
        p.update(lo=lo, hi=hi, sense=sense.to(torch.int8))
    p.update(m=m, n=n, row=row[order], col=col[order], val=val[order], t_row=col, t_col=row, t_val=val, x=x, y=y, z=z)
    p["b"] = _mul(p["row"], p["col"], p["val"], x, m) + b0
    p["c"] = _mul(col, row, val, y, n) + z
    p["gen"] = g
    return p


def _sizes(case):
    """Rows and columns of a batch's instances: log-uniform over [m_lo, m_hi], in an order of their own."""
    B = case["count"]
    if case["kind"] == "unrolled":
        return np.full(B, case["m"]), np.full(B, case["n"])
    q = (np.arange(B) + 0.5) / B
    ms = np.rint(case["m_lo"] * (case["m_hi"] / case["m_lo"]) ** q).astype(np.int64)
    ms = np.random.RandomState(B).permutation(ms)
    return ms, np.rint(2.5 * ms).astype(np.int64)


def _scaling(p):
    """Ten infinity-norm passes and one 1-norm pass of |A|: the factors of a PDHG solve's scaled LP."""
    dr = torch.ones(p["m"], device=DEV, dtype=F64)
    dc = torch.ones(p["n"], device=DEV, dtype=F64)
    for k in range(RUIZ + 1):
        red = "max" if k < RUIZ else "sum"
        sr = dr * _by_row(p["row"], p["val"].abs() * dc[p["col"]], p["m"], red)
        sc = dc * _by_row(p["t_row"], p["t_val"].abs() * dr[p["t_col"]], p["n"], red)
        dr = dr * torch.where(sr > 0, 1.0 / sr.sqrt(), 1.0)
        dc = dc * torch.where(sc > 0, 1.0 / sc.sqrt(), 1.0)
    return dr, dc


def _warm_point(p):
    """A point as a PDHG solve to 1e-4 leaves it: the planted optimum with errors of that size."""
    g = p["gen"]
    noise = [1e-4 * torch.randn(k, generator=g, device=DEV, dtype=F64) for k in (p["n"], p["m"], p["n"])]
    return (p["x"] + noise[0]).clamp(min=0.0), p["y"] + noise[1], (p["z"] + noise[2]).clamp(min=0.0)


def _shape(case) -> dict:
    """Kernel shapes for the large block-angular LPs, as the autotuner picks them; defaults elsewhere."""
    if case["lp"] == "block" and case["nblocks"] * case["bn"] >= 500000:
        return dict(spmv_kind=3, tile_nnz=8192, tile_rows=512, short_row=32, tile_nnz_at=4096, tile_rows_at=512,
                    short_row_at=32)
    return {}


class _Point:
    """What ipm_warm reads of a Solution."""

    def __init__(self, x, y, z, d_row, d_col):
        self.x, self.y, self.z, self.d_row, self.d_col = x, y, z, d_row, d_col


def prepare(case, seed):
    p = _problem(case, seed)
    A = _Csr((p["m"], p["n"]), p["row"], p["col"], p["val"])
    AT = _Csr((p["n"], p["m"]), p["t_row"], p["t_col"], p["t_val"])
    b, c = p["b"].cpu().numpy(), p["c"].cpu().numpy()
    s = dict(case=case)
    if case["kind"] in ("batch", "unrolled"):
        ro, co = p["row_off"].cpu().numpy(), p["col_off"].cpu().numpy()
        s["batch"] = P.DeviceBatch(A, AT, b, c, ro, co, co * case.get("per_col", 4), DEV)
        if case["kind"] == "unrolled":
            s["map"] = P.UnrolledMap(s["batch"], K=case["K"], ckpt_every=case["ckpt"], precision=case["precision"])
            s["w"] = torch.randn(p["n"], generator=p["gen"], device=DEV, dtype=F64)
            s["c"], s["b"] = p["c"], p["b"]
        return s
    host = [None if p[k] is None else p[k].cpu().numpy() for k in ("lo", "hi", "sense")]
    s["lp"] = P.DeviceLP(A, AT, b, c, DEV, *host)
    if case["kind"].startswith("ipm"):
        dr, dc = _scaling(p)
        s["d"] = (dr, dc)
        if case["kind"] == "ipm_warm":
            s["point"] = _Point(*_warm_point(p), dr, dc)
    return s


# ---------------------------------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------------------------------
def run(s):
    case = s["case"]
    if case["kind"] == "ipm_cold":
        r = P.ipm_solve(s["lp"], *s["d"], max_iter=case["steps"])
        return [r.x, r.y, r.z]
    if case["kind"] == "ipm_warm":
        r = P.ipm_warm(s["lp"], s["point"], max_iter=case["steps"])
        return [r.x, r.y, r.z]
    if case["kind"] == "unrolled":
        c, b = s["c"].detach().requires_grad_(), s["b"].detach().requires_grad_()
        xK = s["map"].apply(c, b)
        xK.backward(s["w"])
        out = [xK.detach(), c.grad, b.grad]
    else:
        if case["kind"] == "batch":
            r = P.solve_batched(s["batch"], 1e-6, case["precision"], max_iter=case["iters"])
        else:
            r = P.solve(s["lp"], 1e-6, case["precision"], max_iter=case["iters"], **_shape(case))
        out = [r.x, r.y, r.z] + ([r.r_p, r.r_d] if case["precision"] == "fp64" else [])
    return out if case["precision"] == "fp64" else [v.float() for v in out]


# ---------------------------------------------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------------------------------------------
def _nnz(case):
    if case["kind"] in ("batch", "unrolled"):
        ms, ns = _sizes(case)
        return int(ms.sum()), int(ns.sum()), int(ns.sum()) * case.get("per_col", 4)
    if case["lp"] == "block":
        n = case["nblocks"] * case["bn"]
        return case["nblocks"] * case["bm"] + case["nlink"], n, 6 * n + case["nlink"] * case["link_nnz"]
    if case["lp"] == "uniform":
        return case["m"], case["n"], case["n"] * min(case["per_col"], case["m"])
    k = np.arange(2, min(2000, case["m"]) + 1, dtype=np.float64)
    q = k ** -2.1423
    return case["m"], case["n"], int(case["n"] * float((k * q).sum() / q.sum()))


def work(case):
    m, n, nnz = _nnz(case)
    lp = 2 * (12 * nnz) + 4 * (m + n) + 8 * (m + n)  # A and A^T, b and c, read once
    if case["kind"].startswith("ipm"):
        k = case["steps"]
        # a Newton step: the normal matrix (a multiply-add for each pair of entries of a column), its Cholesky factor
        # (m^3 / 3), two solves with it and the products with A and A^T; the factor written and read by the solves
        pairs = nnz * nnz / n
        fl = k * (2 * pairs / 2 + m ** 3 / 3 + 4 * 2 * m * m + 8 * 2 * nnz)
        return {"bytes": lp + 8 * (m + 2 * n) + k * (3 * 8 * m * m / 2 + 4 * 12 * nnz), "flops": fl}
    vs, ts = VALUE_BYTES[case["precision"]], STATE_BYTES[case["precision"]]
    ib = 4 if case["kind"] == "solve" else 2  # a column index: local in a batch
    sweep = 2 * nnz * (vs + ib)               # both copies of the stored matrix
    iters = case.get("K") or case["iters"]
    step = sweep + ts * (6 * n + 4 * m)       # and the vectors of an iteration
    evals = -(-iters // EVAL_EVERY)
    total = lp + POWER_ITERS * sweep + iters * step
    fl = 4 * nnz * (POWER_ITERS + iters)
    if case["kind"] == "unrolled":            # the reverse sweep recomputes the forward one
        total += 2 * iters * step + 8 * (2 * n + m)
        fl += 2 * 4 * nnz * iters
    else:
        total += evals * 2 * 12 * nnz + 8 * (3 * n + 2 * m)
        fl += evals * 4 * nnz
    return {"bytes": total, "flops": fl}


# ---------------------------------------------------------------------------------------------------------------
# the same results in 64 bits
# ---------------------------------------------------------------------------------------------------------------
class _Inst:
    """Sums and expansions over the instances of a block-diagonal LP (one instance: the whole LP)."""

    def __init__(self, p):
        self.one = "row_off" not in p
        if not self.one:
            ro, co = p["row_off"], p["col_off"]
            self.B = ro.numel() - 1
            ids = torch.arange(self.B, device=DEV)
            self.idx = {p["m"]: torch.repeat_interleave(ids, ro.diff()), p["n"]: torch.repeat_interleave(ids, co.diff())}
            self.nn = co.diff().to(F64)
            assert p["m"] != p["n"]
        else:
            self.B, self.nn = 1, torch.full((1,), float(p["n"]), device=DEV, dtype=F64)

    def sum(self, v):
        if self.one:
            return v.sum().reshape(1)
        return torch.zeros(self.B, device=DEV, dtype=v.dtype).index_add_(0, self.idx[v.numel()], v)

    def norm(self, v):
        return self.sum(v * v).sqrt()

    def to(self, s, size):
        return s.expand(size) if self.one else s[self.idx[size]]


def _pdhg(p, iters, precision, eps=None, grad_w=None):
    """The solve's iteration in float64.  eps: stop and evaluate as the solve does; grad_w: the unrolled map and its
    gradients for the loss w . x_K, the schedule held constant."""
    I, m, n = _Inst(p), p["m"], p["n"]
    row, col, tr, tc = p["row"], p["col"], p["t_row"], p["t_col"]
    dr, dc = _scaling(p)
    val, tval = dr[row] * p["val"] * dc[col], dc[tr] * p["t_val"] * dr[tc]
    if precision == "bf16":  # the matrix such a solve iterates on
        val, tval = val.float().bfloat16().to(F64), tval.float().bfloat16().to(F64)

    def A(v):
        return torch.zeros(m, device=DEV, dtype=F64).index_add(0, row, val * v[col])

    def AT(v):
        return torch.zeros(n, device=DEV, dtype=F64).index_add(0, tr, tval * v[tc])

    def true_A(v):
        return _mul(row, col, p["val"], v, m)

    def true_AT(v):
        return _mul(tr, tc, p["t_val"], v, n)

    v = I.to(1.0 / I.nn.sqrt(), n)
    hist = []
    for k in range(POWER_ITERS + 1):
        av = A(v)
        hist.append(I.norm(av))
        if k < POWER_ITERS:
            u = AT(av)
            v = u / I.to(I.norm(u), n)
    h = hist[-1]
    eta = torch.where((h - hist[-11]).abs() > 1e-3 * h, 0.95, 0.95 / h)
    bb, cc = p["b"], p["c"]
    if grad_w is not None:
        bb, cc = bb.clone().requires_grad_(), cc.clone().requires_grad_()
    ct, bt = dc * cc, dr * bb
    om = I.norm(ct.detach()) / I.norm(bt.detach())
    lo = p["lo"] / dc if p["lo"] is not None else None
    hi = p["hi"] / dc if p["hi"] is not None else None
    sense = p["sense"]
    bnorm, cnorm = I.norm(p["b"]), I.norm(p["c"])
    zero_n, zero_m = torch.zeros(n, device=DEV, dtype=F64), torch.zeros(m, device=DEV, dtype=F64)
    x0, y0, u, v = zero_n, zero_m, zero_n, zero_m  # the anchor and the state relative to it
    rc, rb = ct, bt                               # the anchor's residuals, formed on the unrounded matrix
    k = torch.zeros(I.B, device=DEV, dtype=F64)
    R0, Rp = torch.zeros_like(k), torch.full_like(k, math.inf)
    live = torch.ones(I.B, device=DEV, dtype=torch.bool)
    out = None
    for t in range(1, iters + 1):
        tau, sig = (eta / om).detach(), (eta * om).detach()
        w = (k + 1) / (k + 2)
        g = u - I.to(tau, n) * (rc - AT(v))
        if lo is None:
            uh = torch.maximum(g, -x0)
        else:
            uh = torch.minimum(torch.maximum(g, lo - x0), hi - x0)
        vh = v + I.to(sig, m) * (rb - A(2.0 * uh - u))
        if sense is not None:
            vh = torch.where(sense == 1, torch.maximum(vh, -y0), torch.where(sense == 2, torch.minimum(vh, -y0), vh))
        with torch.no_grad():
            first = k == 0
            ev = t % EVAL_EVERY == 0 or (t == iters and grad_w is None)
            if ev or bool(first.any()):
                R = (om * I.norm(u - uh) ** 2 + I.norm(v - vh) ** 2 / om).sqrt()
                R0 = torch.where(first, R, R0)
        xh, yh = x0 + uh, y0 + vh
        u, v = I.to(w, n) * (2.0 * uh - u), I.to(w, m) * (2.0 * vh - v)
        k = k + 1
        if grad_w is not None and t == iters:
            xk = dc * xh
            gc, gb = torch.autograd.grad((xk * grad_w).sum(), [cc, bb])
            return [xk.detach(), gc, gb]
        if not ev:
            continue
        with torch.no_grad():
            if grad_w is None:
                x, y = dc * xh, dr * yh
                rp, red = p["b"] - true_A(x), p["c"] - true_AT(y)
                if sense is not None:
                    rp = torch.where(sense == 1, rp.clamp(min=0), torch.where(sense == 2, rp.clamp(max=0), rp))
                if lo is None:
                    z, bterm = red.clamp(min=0), torch.zeros_like(red)
                else:
                    lf, hf = p["lo"].isfinite(), p["hi"].isfinite()
                    z = torch.where(lf & hf, red, torch.where(lf, red.clamp(min=0), torch.where(hf, red.clamp(max=0), 0.0)))
                    bterm = torch.where(lf, p["lo"], 0.0) * z.clamp(min=0) + torch.where(hf, p["hi"], 0.0) * z.clamp(max=0)
                new = [x, y, z, rp, red - z]
                out = new if out is None else [torch.where(I.to(live, a.numel()), a, o) for a, o in zip(new, out)]
                po, do = I.sum(p["c"] * x), I.sum(p["b"] * y) + I.sum(bterm)
                done = (I.norm(rp) <= eps * (1 + bnorm)) & (I.norm(red - z) <= eps * (1 + cnorm)) & \
                    ((po - do).abs() <= eps * (1 + po.abs() + do.abs()))
                live = live & ~done
                if t == iters or not bool(live.any()):
                    return out
            again = (R <= 0.2 * R0) | ((R <= 0.8 * R0) & (R > Rp)) | (k >= 0.36 * t)
            dx, dy = I.norm(uh), I.norm(vh)
            move = again & (dx > 1e-10) & (dy > 1e-10)
            om = torch.where(move, (dy / dx * om).clamp(min=1e-300).sqrt(), om)
            Rp = torch.where(again, math.inf, R)
            k = torch.where(again, 0.0, k)
        an, am = I.to(again, n), I.to(again, m)
        x0, y0 = torch.where(an, xh, x0), torch.where(am, yh, y0)
        u, v = torch.where(an, 0.0, u), torch.where(am, 0.0, v)
        if precision == "bf16":
            rb = torch.where(am, dr * (bb - true_A(dc * x0)), rb)
            rc = torch.where(an, dc * (cc - true_AT(dr * y0)), rc)
        else:
            rb, rc = torch.where(am, bt - A(x0), rb), torch.where(an, ct - AT(y0), rc)
    return out


def _centered(x, z, mu_min=1e-6, delta=1e-4, alpha=1e-6):
    """Algorithm 1 on a scaled point."""
    mu = max(float(x @ z) / x.numel(), mu_min)
    xl, zl = x.clamp(min=alpha), z.clamp(min=alpha)
    xf = xl < zl
    a, b = torch.where(xf, xl, zl), torch.where(xf, zl, xl)

    def pull(v, to):
        return torch.minimum(torch.maximum(to, v - delta), v + delta)

    a = pull(a, mu / b)
    b = pull(b, mu / a)
    return torch.where(xf, a, b), torch.where(xf, b, a)


def _newton(A, b, c, x, y, z, steps, tol=1e-8):
    """Mehrotra's predictor-corrector; returns the point and the first step length."""
    first = None
    for _ in range(steps):
        rb, rc = b - A @ x, c - A.T @ y - z
        px, dy_ = float(c @ x), float(b @ y)
        rel = max(float(rb.norm() / (1 + b.norm())), float(rc.norm() / (1 + c.norm())),
                  abs(px - dy_) / (1 + abs(px) + abs(dy_)))
        if rel <= tol:
            break
        mu = float(x @ z) / x.numel()
        d = x / z
        L = torch.linalg.cholesky((A * d) @ A.T)

        def direction(rxz):
            t = rxz / z - d * rc
            dy = torch.cholesky_solve((rb - A @ t)[:, None], L)[:, 0]
            v = A.T @ dy
            return d * v + t, dy, rc - v

        def room(v, dv):
            q = torch.where(dv < 0, -v / dv, math.inf)
            return float(q.min())

        dx, dy, dz = direction(-x * z)
        ap, ad = min(1.0, room(x, dx)), min(1.0, room(z, dz))
        sigma = (float((x + ap * dx) @ (z + ad * dz)) / x.numel() / mu) ** 3
        dx, dy, dz = direction(sigma * mu - x * z - dx * dz)
        ap, ad = min(1.0, 0.9995 * room(x, dx)), min(1.0, 0.9995 * room(z, dz))
        first = min(ap, ad) if first is None else first
        x, y, z = x + ap * dx, y + ad * dy, z + ad * dz
    return x, y, z, first


def exact(case, seed):
    p = _problem(case, seed)
    if case["kind"] in ("solve", "batch"):
        return _pdhg(p, case["iters"], case["precision"], eps=1e-6)[:5 if case["precision"] == "fp64" else 3]
    if case["kind"] == "unrolled":
        w = torch.randn(p["n"], generator=p["gen"], device=DEV, dtype=F64)
        return _pdhg(p, case["K"], case["precision"], grad_w=w)
    dr, dc = _scaling(p)
    A = torch.zeros((p["m"], p["n"]), device=DEV, dtype=F64)
    A[p["row"], p["col"]] = dr[p["row"]] * p["val"] * dc[p["col"]]
    b, c = dr * p["b"], dc * p["c"]
    if case["kind"] == "ipm_cold":
        L = torch.linalg.cholesky(A @ A.T)
        x = A.T @ torch.cholesky_solve(b[:, None], L)[:, 0]
        y = torch.cholesky_solve((A @ c)[:, None], L)[:, 0]
        z = c - A.T @ y
        x, z = x + max(-1.5 * float(x.min()), 0.0), z + max(-1.5 * float(z.min()), 0.0)
        xz, sx, sz = float(x @ z), float(x.sum()), float(z.sum())
        x, y, z, _ = _newton(A, b, c, x + 0.5 * xz / sz, y, z + 0.5 * xz / sx, case["steps"])
    else:
        x, y, z = _warm_point(p)
        xs, zs = _centered(x / dc, z * dc)
        alpha = 1e-6
        for _ in range(13):
            x, yy, z, first = _newton(A, b, c, xs, y / dr, zs, case["steps"])
            if first is None or first >= 1e-6:
                break
            alpha *= 10.0
            xs, zs = xs.clamp(min=alpha), zs.clamp(min=alpha)
        y = yy
    return [dc * x, dr * y, z / dc]
