"""LPs that one workgroup holds (k_small_iters, k_small_power, k_small_scale):
every precision and form against the tile kernels and the oracle, and traced or
timed solves against the plain one."""
import numpy as np
import pytest

import lpgen
import oracle
from oracle.pdhg import OracleOptions
from test_gpu_layout import _small

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2603_03150_amd")
torch = pytest.importorskip("torch")

PRECS = ["fp64", "fp32", "bf16", "fp32acc32", "fp32a"]


def _np(t):
    return t.detach().cpu().numpy()


def _lp(general, seed=0):
    return lpgen.general_cfg1(seed) if general else lpgen.cfg1(seed)


@pytest.mark.parametrize("general", [False, True])
@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("kw", [dict(trace_iters=200), dict(trace_iters=5), dict(kernel_timing=1),
                                dict(kernel_timing=2), dict(trace_iters=70, kernel_timing=1)])
def test_traced_and_timed_solves_are_the_plain_solve(prec, general, kw):
    dlp = P.DeviceLP.from_lp(_lp(general))
    for T, E in ((200, 64), (37, 64), (66, 3), (4, 1), (9, 2)):
        a = P.solve(dlp, 1e-14, prec, max_iter=T, eval_every=E)
        b = P.solve(dlp, 1e-14, prec, max_iter=T, eval_every=E, **kw)
        assert a.status == b.status and a.info["iters"] == b.info["iters"] == T
        assert a.info["restarts"] == b.info["restarts"] and a.info["omega"] == b.info["omega"]
        for k in ("x", "y", "z", "r_p", "r_d"):
            assert torch.equal(getattr(a, k), getattr(b, k)), (k, T, E)
        if "kernel_timing" in kw:
            n = 256 if kw["kernel_timing"] == 2 else T
            assert b.info["n_primal"] == b.info["n_dual"] == n
            assert b.info["ms_primal"] > 0 and b.info["ms_dual"] > 0
        if kw.get("trace_iters", 0) >= T:  # the last iteration's projected point is the evaluated one
            assert np.allclose(_np(b.trace["xhat"][T - 1] * b.d_col), _np(b.x), rtol=1e-6, atol=1e-6)


def test_the_autotuner_times_what_a_small_lp_runs():
    # one workgroup's iteration is several times as fast as any pair of tile launches at this size
    dlp = P.DeviceLP.from_lp(lpgen.cfg1(0))
    best = P.autotune(dlp, "fp32", iters=64)
    shape = {k: v for k, v in best.items() if k not in ("ms_per_iter", "cache_hit")}
    assert shape["spmv_kind"] == 0
    a = P.solve(dlp, 1e-14, "fp32", max_iter=150)
    b = P.solve(dlp, 1e-14, "fp32", max_iter=150, **shape)
    assert torch.equal(a.x, b.x) and torch.equal(a.y, b.y)
    timed = P.solve(dlp, 1e-14, "fp32", max_iter=150, kernel_timing=2).info
    assert best["ms_per_iter"] <= 1.5 * (timed["ms_primal"] + timed["ms_dual"])


def _rel(a, b):
    return float(np.linalg.norm(a - b)) / max(1.0, float(np.linalg.norm(b)))


def _gen(lp):
    return dict(lo=lp.lo, hi=lp.hi, sense=lp.sense) if lp.general else {}


# The same tiles as the default shape's on an LP of fewer than 511 rows and columns, but named by the caller: the tile
# kernels in their sorted layout.
TILES = dict(tile_rows=511)


@pytest.mark.parametrize("make", [lambda: lpgen.cfg1(0), lambda: lpgen.tiny(6, 15, 3, 2), lambda: lpgen.general_cfg1(0),
                                  lambda: lpgen.general_tiny(12, 30, 3, 1)])
@pytest.mark.parametrize("kw", [TILES, dict(TILES, gather_order=1), dict(tile_nnz=256, tile_rows=64), dict(spmv_kind=2)])
def test_tile_kernels_on_a_small_lp_follow_the_oracle(make, kw):
    lp, T = make(), 100
    sol = P.solve(P.DeviceLP.from_lp(lp), 1e-14, "fp64", trace_iters=T, max_iter=T, **kw)
    ref = oracle.solve(lp.A, lp.AT, lp.b, lp.c, 1e-14, opts=OracleOptions(max_iter=T), trace_iters=T, **_gen(lp))
    assert sol.status == ref.status and abs(sol.info["sigma_hat"] - ref.sigma_hat) <= 1e-12 * ref.sigma_hat
    for t in range(1, min(T, ref.iters) + 1):
        for key, r in zip(("x", "y", "xhat", "yhat"), ref.trace[t]):
            assert _rel(_np(sol.trace[key][t - 1]), r) <= 1e-10, (t, key)


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("kw", [dict(), TILES, dict(spmv_kind=2), dict(tile_nnz=1024)])
def test_standard_bounds_and_senses_are_bitwise_the_standard_form(prec, kw):
    lp = lpgen.cfg1(0)
    g = P.DeviceLP(lp.A, lp.AT, lp.b, lp.c, lo=np.zeros(lp.n), hi=np.full(lp.n, np.inf),
                   sense=np.zeros(lp.m, dtype=np.int8))
    a = P.solve(P.DeviceLP.from_lp(lp), 1e-14, prec, max_iter=300, **kw)
    b = P.solve(g, 1e-14, prec, max_iter=300, **kw)
    assert a.info["iters"] == b.info["iters"] and a.info["restarts"] == b.info["restarts"]
    for k in ("x", "y", "z", "r_p", "r_d"):
        assert torch.equal(getattr(a, k), getattr(b, k)), k


@pytest.mark.parametrize("prec", PRECS)
def test_named_kernels_of_a_small_lp_agree_bitwise(prec):
    # the persistent grid and both orders of the loads add the same tiles in the same order
    dlp = P.DeviceLP.from_lp(lpgen.cfg1(0))
    a, b, c = (P.solve(dlp, 1e-14, prec, max_iter=200, **kw)
               for kw in (TILES, dict(spmv_kind=2), dict(TILES, gather_order=1)))
    assert torch.equal(a.x, b.x) and torch.equal(a.y, b.y)
    assert torch.equal(a.x, c.x) and torch.equal(a.y, c.y)


@pytest.mark.parametrize("general", [False, True])
@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("name", ["one", "empty_rows_and_columns", "lanes_8", "lanes_4", "lanes_2", "two_rows",
                                  "rows_2048", "row_192"])
def test_one_workgroup_against_the_tile_kernels(name, prec, general):
    """The same iteration with a row's terms added in another order.  One epoch (no restart before 64): the iteration
    is nonexpansive, so the points differ by at most the sum of what each iteration's stores and sums round (2 ulp of
    a float32, or one for each term of the longest row where sums are float32 too) and of what the two step sizes
    differ by; a factor of 4 for the primal weight's norm."""
    lp, T = _small(name), 60
    if general:
        lp = lpgen.general_from_matrix(lp.A, lp.AT, lpgen.rng_for(81, len(name)))
    dlp = P.DeviceLP.from_lp(lp)
    a = P.solve(dlp, 1e-14, prec, max_iter=T)
    b = P.solve(dlp, 1e-14, prec, max_iter=T, tile_nnz=1024)
    longest = int(max(np.diff(lp.A.indptr).max(), np.diff(lp.AT.indptr).max()))
    ulp = 2.0 ** -53 if prec in ("fp64", "fp32a") else 2.0 ** -24
    terms = longest + 4 if prec in ("fp32acc32", "fp64", "fp32a") else 2
    # the power iteration stores its vectors, and each of its steps rounds them once
    dsig = abs(a.info["sigma_hat"] - b.info["sigma_hat"]) / b.info["sigma_hat"]
    assert dsig <= 2 * 101 * (longest if ulp < 1e-10 else 1) * ulp
    deta = abs(a.info["eta"] - b.info["eta"]) / b.info["eta"]
    tol = 4 * T * (deta + terms * ulp)
    assert a.info["restarts"] == b.info["restarts"] == 0
    scale = float(torch.sqrt((b.x / b.d_col).square().sum() + (b.y / b.d_row).square().sum()))
    for u, v, d in ((a.x, b.x, b.d_col), (a.y, b.y, b.d_row)):
        assert float(torch.linalg.norm((u - v) / d)) <= tol * max(scale, 1e-300)
