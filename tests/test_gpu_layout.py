"""The layouts and workgroup classes of instances held by one workgroup.

Shapes at the edges: one row or column, columns and rows without entries,
sizes beside multiples of a wave and of three, a row and a column too long for
the level layout, more rows than it takes, and more entries than LDS holds.
FP64 is compared with the oracle at the tolerances of the other per-iterate
tests (1e-10 over at most 150 iterations, 1e-8 for gradients).  An instance's
bits must not depend on the workgroup that held it: alone, in a batch of more
instances than compute units (other classes), and under a launch split.
"""
import numpy as np
import pytest

import lpgen
import oracle
from oracle.pdhg import OracleOptions

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2603_03150_amd")
torch = pytest.importorskip("torch")


def _np(t):
    return t.detach().cpu().numpy()


def _rel(a, b):
    return float(np.linalg.norm(a - b)) / max(1.0, float(np.linalg.norm(b)))


def _planted(name, m, counts, extra=None):
    """counts[j] distinct uniform rows in column j; extra(j) more of them."""
    rng = lpgen.rng_for(77, len(name), m, len(counts))
    cols = []
    for j, k in enumerate(counts):
        rows = set(rng.choice(m, size=min(int(k), m), replace=False).tolist())
        if extra is not None:
            rows |= set(extra(j))
        cols.append(sorted(rows))
    cnt = np.array([len(r) for r in cols], dtype=np.int64)
    rows = np.array([i for r in cols for i in r], dtype=np.int64)
    return lpgen.planted_from_columns(m, cnt, rows, rng.standard_normal(rows.size), rng, name=name)


def _shape(name):
    rng = lpgen.rng_for(78, len(name))
    if name == "one":
        return _planted(name, 1, [1])
    if name == "one_row":
        return _planted(name, 1, [1] * 65)
    if name == "ragged_63":  # columns and rows without entries
        return _planted(name, 63, rng.integers(0, 4, size=64))
    if name == "ragged_193":  # past three columns to a thread of one wave
        return _planted(name, 65, rng.integers(0, 8, size=193))
    if name == "wide_3073":  # past three columns to a thread of 1,024
        return _planted(name, 1025, rng.integers(1, 6, size=3073))
    if name == "long_row":  # 1,100 entries: CSR order
        return _planted(name, 70, [3] * 1100, extra=lambda j: [0])
    if name == "long_column":
        return _planted(name, 1030, [4] * 2000, extra=lambda j: range(1030) if j == 7 else [])
    if name == "many_rows":  # more rows than the level layout takes
        return _planted(name, 8300, [60] * 300)
    if name == "partial":  # a matrix that LDS holds in part
        return _planted(name, 300, [24] * 2500)
    raise ValueError(name)


NAMES = ["one", "one_row", "ragged_63", "ragged_193", "wide_3073", "long_row", "long_column", "many_rows", "partial"]


@pytest.mark.parametrize("name", NAMES)
def test_batched_shape_matches_oracle_and_bits_do_not_depend_on_the_class(name):
    lp, T = _shape(name), 70
    alone = P.solve_batched(P.DeviceBatch.from_lps([lp]), 1e-14, "fp64", max_iter=T)
    ref = oracle.solve(lp.A, lp.AT, lp.b, lp.c, 1e-14, opts=OracleOptions(max_iter=T))
    assert alone.infos[0]["iters"] == ref.iters and alone.infos[0]["restarts"] == ref.restarts
    assert _rel(_np(alone.x), ref.meas.x) <= 1e-10
    assert _rel(_np(alone.y), ref.meas.y) <= 1e-10
    fill = [lpgen.cfg4_instance(2000 + i, m) for i, m in enumerate([20, 90, 300] * 100)]
    batch = P.DeviceBatch.from_lps([lp] + fill)
    for prec in ("fp64", "fp32", "fp32acc32", "bf16"):
        one = P.solve_batched(P.DeviceBatch.from_lps([lp]), 1e-14, prec, max_iter=T)
        for split in (0, 1000):
            many = P.solve_batched(batch, 1e-14, prec, max_iter=T, batch_split=split).split(batch, 0)
            assert np.array_equal(_np(one.x), _np(many["x"])), (prec, split)
            assert np.array_equal(_np(one.y), _np(many["y"])), (prec, split)


@pytest.mark.parametrize("name", NAMES)
def test_unrolled_shape_matches_oracle_and_bits_do_not_depend_on_the_class(name):
    lp, K = _shape(name), 65
    w = lpgen.rng_for(79, len(name)).standard_normal(lp.c.size)

    def run(lps, prec):
        batch = P.DeviceBatch.from_lps(lps)
        umap = P.UnrolledMap(batch, K=K, ckpt_every=32, precision=prec)
        c, b = batch.lp.c.clone(), batch.lp.b.clone()
        xK, tape = umap.forward_raw(c, b)
        g = torch.zeros_like(c)
        g[:w.size] = torch.tensor(w, device="cuda")
        gc, gb = umap.backward_raw(c, b, tape, g)
        n, m = lp.c.size, lp.b.size
        return _np(xK)[:n], _np(gc)[:n], _np(gb)[:m]

    xK, gc, gb = run([lp], "fp64")
    rc, rb, rx, _ = oracle.unrolled_grad(lp.A, lp.b, lp.c, K, w, OracleOptions())
    assert _rel(xK, rx) <= 1e-10
    assert _rel(gc, rc) <= 1e-8
    assert _rel(gb, rb) <= 1e-8
    fill = [lpgen.cfg4_instance(2000 + i, m) for i, m in enumerate([20, 90, 300] * 100)]
    for prec in ("fp64", "fp32", "bf16"):
        for a, b in zip(run([lp], prec), run([lp] + fill, prec)):
            assert np.array_equal(a, b), prec


def _small(name):
    rng = lpgen.rng_for(80, len(name))
    if name == "one":
        return _planted(name, 1, [1])
    if name == "empty_rows_and_columns":
        return _planted(name, 40, rng.integers(0, 3, size=64))
    if name == "lanes_8":  # a row to eight lanes up to 128 of them, with long rows
        return _planted(name, 128, rng.integers(3, 9, size=130))
    if name == "lanes_4":
        return _planted(name, 129, [4] * 257)
    if name == "lanes_2":
        return _planted(name, 257, [4] * 513)
    if name == "two_rows":  # more columns than threads
        return _planted(name, 513, [3] * 1025)
    if name == "rows_2048":
        return _planted(name, 2048, [2] * 2048)
    if name == "scaling_outside":  # fits the iterations' LDS but not the scaling's
        return _planted(name, 2048, [3] * 1300 + [2] * 748)
    if name == "rows_2049":  # past the one workgroup's rows
        return _planted(name, 2049, [2] * 1500)
    if name == "row_192":
        return _planted(name, 30, [2] * 191 + [0], extra=lambda j: [5])
    if name == "row_193":  # past its longest row
        return _planted(name, 30, [2] * 193, extra=lambda j: [5])
    raise ValueError(name)


@pytest.mark.parametrize("general", [False, True])
@pytest.mark.parametrize("name", ["one", "empty_rows_and_columns", "lanes_8", "lanes_4", "lanes_2", "two_rows",
                                  "rows_2048", "scaling_outside", "rows_2049", "row_192", "row_193"])
def test_small_lp_in_one_workgroup_matches_oracle(name, general):
    lp = _small(name)
    kw = {}
    if general:
        lp = lpgen.general_from_matrix(lp.A, lp.AT, lpgen.rng_for(81, len(name)))
        kw = dict(lo=lp.lo, hi=lp.hi, sense=lp.sense)
    for T in (1, 2, 3, 64, 66, 67, 130):  # blocks of 64 with and without iterations between the first and last
        sol = P.solve(P.DeviceLP.from_lp(lp), 1e-14, "fp64", max_iter=T)
        ref = oracle.solve(lp.A, lp.AT, lp.b, lp.c, 1e-14, opts=OracleOptions(max_iter=T), **kw)
        assert sol.info["iters"] == ref.iters and sol.info["restarts"] == ref.restarts, T
        assert abs(sol.info["sigma_hat"] - ref.sigma_hat) <= 1e-12 * ref.sigma_hat
        assert _rel(_np(sol.x), ref.meas.x) <= 1e-10, T
        assert _rel(_np(sol.y), ref.meas.y) <= 1e-10, T


# What the device check of a batch finds, each on a batch with more rows than
# a chunk's LDS holds, most of them without entries.
@pytest.mark.parametrize("what,code,text", [
    ("nothing", 0, ""),
    ("decreasing", -2, "A row pointer decreases at row 2"),
    ("decreasing_t", -2, "A^T row pointer decreases at row 2"),
    ("end", -2, "must start at 0 and end at nnz"),
    ("nnz_off", -2, "nnz_off does not match the row pointers at instance 1"),
    ("column", -2, "column index out of range"),
    ("nan", -7, "NaN or Inf"),
    ("inf_b", -7, "NaN or Inf"),
    ("transpose", -3, "does not match"),
])
def test_batch_check_finds(what, code, text):
    lps = [_planted("sparse", 5000, [2] * 60), lpgen.cfg4_instance(1, 40), _planted("sparse2", 4000, [3] * 30)]
    batch = P.DeviceBatch.from_lps(lps)
    lp = batch.lp
    if what == "decreasing":
        lp.a_rowptr[2], lp.a_rowptr[3] = 50, 10
    elif what == "decreasing_t":
        lp.at_rowptr[2], lp.at_rowptr[3] = 50, 10
    elif what == "end":
        lp.a_rowptr[-1] += 1
    elif what == "nnz_off":
        batch.nnz_off[1] += 1
    elif what == "column":
        lp.at_col[7] = -1
    elif what == "nan":
        lp.at_val[100] = float("nan")
    elif what == "inf_b":
        lp.b[3] = float("inf")
    elif what == "transpose":
        lp.a_val[100] *= 1.0 + 1e-6
    if code == 0:
        assert P.solve_batched(batch, 1e-14, "fp32", max_iter=3).infos[0]["iters"] == 3
        return
    with pytest.raises(P.MipdhgError) as e:
        P.solve_batched(batch, 1e-4, "fp32", max_iter=3)
    assert e.value.code == code and text in str(e.value), str(e.value)


def _rests(name):
    rng = lpgen.rng_for(82, len(name))
    if name == "rows_24":  # at the line for four- and two-byte values
        return _planted(name, 60, [12] * 120)
    if name == "rests_0_to_9":  # rows of 12 to 34 entries, every remainder past the registers' 16
        return _planted(name, 23, [1] * 60, extra=lambda j: [i for i in range(23) if j < 12 + i])
    if name == "columns_14":  # by its columns
        return _planted(name, 90, [14] * 40)
    if name == "two_slots":  # rows past the registers' slots, in two passes
        return _planted(name, 300, rng.integers(20, 40, size=250))
    raise ValueError(name)


@pytest.mark.parametrize("name", ["rows_24", "rests_0_to_9", "columns_14", "two_slots"])
def test_long_rests_match_the_oracle_and_the_short_forms_bits(name):
    # alone these take the form for long rests, among many short rows the other: the same sums in the same order.
    # FP32 against the oracle: 40 iterations from 0, each some four roundings to float32 (6e-8) of matrix and vectors,
    # not amplified by the iteration in its weighted norm: 1e-5, and ten times that for the weights
    lp, T = _rests(name), 40
    ref = oracle.solve(lp.A, lp.AT, lp.b, lp.c, 1e-14, opts=OracleOptions(max_iter=T))
    fill = [_planted("fill", 60, [2] * 150)] * 40 + [_planted("small", 20, [2] * 50)] * 40
    batch = P.DeviceBatch.from_lps([lp] + fill)
    for prec, tol in (("fp64", 1e-10), ("fp32", 1e-4), ("fp32acc32", None), ("bf16", None)):
        one = P.solve_batched(P.DeviceBatch.from_lps([lp]), 1e-14, prec, max_iter=T)
        many = P.solve_batched(batch, 1e-14, prec, max_iter=T).split(batch, 0)
        assert np.array_equal(_np(one.x), _np(many["x"])) and np.array_equal(_np(one.y), _np(many["y"])), prec
        if tol:
            assert _rel(_np(one.x), ref.meas.x) <= tol and _rel(_np(one.y), ref.meas.y) <= tol, prec

    def grads(lps, prec):
        b = P.DeviceBatch.from_lps(lps)
        umap = P.UnrolledMap(b, K=30, ckpt_every=12, precision=prec)
        c, r = b.lp.c.clone(), b.lp.b.clone()
        xK, tape = umap.forward_raw(c, r)
        g = torch.zeros_like(c)
        g[:lp.c.size] = 1.0
        gc, gb = umap.backward_raw(c, r, tape, g)
        return _np(xK)[:lp.c.size], _np(gc)[:lp.c.size], _np(gb)[:lp.b.size]

    for prec in ("fp32", "fp32acc32", "bf16"):
        for a, b in zip(grads([lp], prec), grads([lp] + fill, prec)):
            assert np.array_equal(a, b), prec
