"""LPs that one workgroup holds (k_small_iters, k_small_power, k_small_scale):
every precision and form against the tile kernels and the oracle, and traced or
timed solves against the plain one."""
import numpy as np
import pytest

import lpgen

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
