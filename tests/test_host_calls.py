"""What the library's host code launches, where, and what it waits for, on the
stand-in HIP runtime of hip_host_calls.c (no GPU)."""
import os
import shutil
import subprocess
import sys
import textwrap

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

pytestmark = pytest.mark.skipif(shutil.which("gcc") is None, reason="needs a C compiler")


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    shim = str(tmp_path_factory.mktemp("shim") / "libhiphost.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", shim, os.path.join(HERE, "hip_host_calls.c")], check=True)
    sys.path.insert(0, ROOT)
    from paper_2603_03150_amd import _lib
    if not os.path.exists(_lib.LIB_PATH):
        from paper_2603_03150_amd.build import build
        build()

    def go(code):
        head = f"import sys; sys.path.insert(0, {HERE!r})\nfrom host_calls import *\nh = Host({shim!r})\n"
        p = subprocess.run([sys.executable, "-c", head + textwrap.dedent(code)], capture_output=True, text=True,
                           timeout=120)
        assert p.returncode == 0, p.stdout + p.stderr

    return go


# --- the kernels of an LP that one workgroup holds -------------------------------------------------------------
@pytest.mark.parametrize("opts,small", [
    (dict(), True), (dict(gather_order=1), True), (dict(lanes_a=4, long_row=9), True),
    (dict(tile_nnz=2048, tile_rows=512, short_row=-1), True),  # the defaults by their values
    (dict(tile_nnz_at=2048, tile_rows_at=512, short_row_at=-1), True),
    (dict(spmv_kind=1), False), (dict(spmv_kind=2), False), (dict(tile_nnz=1024), False), (dict(tile_rows=64), False),
    (dict(short_row=32), False), (dict(tile_nnz_at=1024), False), (dict(tile_rows_at=64), False),
    (dict(short_row_at=32), False),
])
def test_a_small_lp_runs_the_kernels_the_caller_asked_for(run, opts, small):
    run(f"""
    assert h.solve(h.lp(20, 60, [3] * 60), h.options(max_iter=128, **{opts!r})) >= 0
    k = h.kernels()
    for name in ("k_small_iters", "k_small_power", "k_small_scale"):
        assert any(name in n for n in k) == {small}, name
    kind = {opts!r}.get("spmv_kind", 0)
    iters = ["k_iter_persist" if kind == 2 else "k_iter_tiled" if kind == 0 else "6k_iterI"]
    assert any(iters[0] in n for n in k), sorted(set(k))
    """)


@pytest.mark.parametrize("opts,launches", [
    (dict(), 2), (dict(use_graph=0), 2), (dict(kernel_timing=1), 2),
    (dict(kernel_timing=2), 3),                # and one for the timing after the solve
    (dict(trace_iters=128), 2 * 62), (dict(trace_iters=3, kernel_timing=1), 2 * 62),
])
def test_a_small_lp_traced_or_timed_is_the_same_solve(run, opts, launches):
    run(f"""
    assert h.solve(h.lp(20, 60, [3] * 60), h.options(max_iter=128, eval_every=64, **{opts!r})) >= 0
    graph = sum(w == "graph" for w, _, _ in h.log())
    k = h.kernels()
    times = 2 if graph else 1  # the graph's launches are noted once
    small = sum("k_small_iters" in n for n in k)
    tiles = sum("k_iter_tiled" in n for n in k)
    if graph:
        assert graph == 2
        small, tiles = small + 1, tiles + 4
    # a block's first and last iteration on the tiles, primal and dual
    assert (small, tiles) == ({launches}, 8), (small, tiles)
    """)


# --- errors -----------------------------------------------------------------------------------------------------
SETUP_CALLS = ("hipStreamCreateWithFlags", "hipStreamBeginCapture", "hipStreamEndCapture", "hipGraphInstantiate",
               "hipHostMalloc", "hipEventCreateWithFlags", "hipMemcpyAsync", "hipGraphLaunch", "hipEventRecord",
               "hipEventSynchronize", "hipFuncSetAttribute")


@pytest.mark.parametrize("opts", [dict(), dict(spmv_kind=2, kernel_timing=1), dict(spmv_kind=3, panel_width=64),
                                  dict(kernel_timing=2)])
def test_an_error_in_a_solve_leaves_nothing_running(run, opts):
    run(f"""
    lp = h.lp(20, 60, [3] * 60)
    o = h.options(max_iter=192, **{opts!r})
    assert h.errors_leave_nothing_running(lambda: h.solve(lp, o, stream=7), {SETUP_CALLS!r}) >= 10
    """)


BATCH_CALLS = ("hipStreamCreateWithFlags", "hipEventCreate", "hipEventCreateWithFlags", "hipEventRecord",
               "hipStreamWaitEvent", "hipFuncSetAttribute", "hipOccupancyMaxActiveBlocksPerMultiprocessor",
               "hipMemcpyAsync", "hipDeviceGetAttribute", "hipEventElapsedTime")


@pytest.mark.parametrize("opts", [dict(), dict(batch_split=400)])
def test_an_error_in_a_batched_solve_leaves_nothing_running(run, opts):
    run(f"""
    # instances of every launch class (more than compute units)
    lps = [(20, 50, [3] * 50)] * 300 + [(200, 500, [4] * 500)] * 2 + [(500, 1500, [4] * 1500), (2000, 5000, [4] * 5000)]
    b, o = h.batch(lps), h.options("fp32", max_iter=64, **{opts!r})
    assert h.errors_leave_nothing_running(lambda: h.solve_batched(b, o, stream=7), {BATCH_CALLS!r}) >= 20
    """)


def test_an_error_in_the_unrolled_map_leaves_nothing_running(run):
    run(f"""
    b, o = h.batch([(20, 50, [3] * 50)] * 3), h.options("fp32")
    assert h.errors_leave_nothing_running(lambda: h.unrolled(b, o, stream=7), {BATCH_CALLS!r}) >= 10
    """)


IPM_CALLS = ("hipMemcpyAsync", "hipMemsetAsync", "hipFuncSetAttribute", "hipStreamSynchronize", "hipLaunchKernel")


@pytest.mark.parametrize("call,start", [("mipdhg_ipm_solve", True), ("mipdhg_ipm_solve", False),
                                        ("mipdhg_ipm_warm", True)])
def test_an_error_in_the_interior_point_method_leaves_nothing_running(run, call, start):
    run(f"""
    lp = h.lp(2, 3, [1, 2, 1])
    nb = C.c_size_t(0)
    assert h.lib.mipdhg_ipm_workspace_size(C.byref(lp), C.byref(nb)) == 0
    ws = h.buf(nb.value)
    # (kernels do not run here: the residuals are zeros and the method ends at its first test)
    assert h.errors_leave_nothing_running(lambda: h.ipm(lp, ws, nb.value, 7, {call!r}, {start}), {IPM_CALLS!r}) >= 10
    """)


# --- the batched solve's streams --------------------------------------------------------------------------------
@pytest.mark.parametrize("opts", [dict(), dict(batch_split=400)])
@pytest.mark.parametrize("masked", [False, True])
def test_a_batch_stays_on_a_stream_with_a_compute_unit_mask(run, opts, masked):
    run(f"""
    lps = [(20, 50, [3] * 50)] * 300 + [(200, 500, [4] * 500)] * 2 + [(500, 1500, [4] * 1500), (2000, 5000, [4] * 5000)]
    b, o = h.batch(lps), h.options("fp32", max_iter=64, **{opts!r})
    h.shim.shim_reset()
    if {masked}:
        h.shim.shim_mask(C.c_void_p(7))
    assert h.solve_batched(b, o, stream=7) >= 0
    on = [s for w, n, s in h.log() if w == "kernel" and "k_batched" in n]
    assert len(on) >= 4 and (set(on) == {{7}}) == {masked}, on
    # otherwise the others' streams start after the caller's work and it waits for them
    waits = [s for w, n, s in h.log() if w == "wait"]
    assert set(on) - {{7}} <= set(waits) and waits.count(7) == len(set(on)) - 1
    """)


@pytest.mark.parametrize("count,m,n,threads", [
    (1, 20, 64, 64), (256, 20, 64, 64), (256, 20, 65, 256),  # no more than compute units: a thread to a column
    (257, 20, 64, 64), (257, 20, 65, 256), (1024, 80, 200, 256), (1025, 80, 200, 64), (1025, 120, 300, 256),
    (11, 65, 45, 256), (300, 65, 45, 256), (1, 100, 256, 256),
])
def test_one_wave_takes_what_256_threads_cannot_hold_at_once(run, count, m, n, threads):
    run(f"""
    b, o = h.batch([({m}, {n}, [4] * {n})] * {count}), h.options("fp32", max_iter=64)
    for call in (h.solve_batched, h.unrolled):
        h.shim.shim_reset()
        assert call(b, o) >= 0
        k = [n for n in h.kernels() if "k_batched" in n or "k_unrolled" in n]
        assert k and all("Li{threads}E" in n for n in k), k
    """)


@pytest.mark.parametrize("n,batched,unrolled", [(257, 512, 1024), (512, 512, 1024), (1024, 512, 1024), (1025, 1024, 1024)])
def test_few_instances_get_about_a_thread_to_a_column(run, n, batched, unrolled):
    run(f"""
    b, o = h.batch([(100, {n}, [4] * {n})] * 3), h.options("fp32", max_iter=64)
    for call, threads in ((h.solve_batched, {batched}), (h.unrolled, {unrolled})):
        h.shim.shim_reset()
        assert call(b, o) >= 0
        k = [n for n in h.kernels() if "k_batched" in n or "k_unrolled" in n]
        assert k and all(f"Li{{threads}}E" in n for n in k), k
    """)


# --- a kept workspace -------------------------------------------------------------------------------------------
def test_a_batch_state_of_the_former_layout_is_refused(run):
    run("""
    b, o = h.batch([(20, 50, [3] * 50)] * 3), h.options("fp32", max_iter=64, batch_block_iters=32)
    nb = C.c_size_t(0)
    assert h.lib.mipdhg_batch_workspace_size(C.byref(b), C.byref(o), C.byref(nb)) == 0
    h.buf = lambda n, got={}, buf=h.buf: got.setdefault(n, buf(n))  # the second call's workspace is the first's
    assert h.solve_batched(b, o) >= 0
    o.resume = 1
    assert h.solve_batched(b, o) >= 0
    hdr = np.ctypeslib.as_array(C.cast(h.buf(nb.value), C.POINTER(C.c_uint64)), (2,))
    kept = hdr.copy()
    hdr[0] = 0x6d69706468672d62  # as written when the vectors lay by row and column
    assert h.solve_batched(b, o) == -1 and b"does not hold the state" in h.lib.mipdhg_last_error()
    hdr[:] = kept
    assert h.solve_batched(b, o) >= 0
    """)


# --- the interior point's triangular solves ---------------------------------------------------------------------
def test_a_triangular_solve_whose_wait_ran_out_is_an_error(run):
    run("""
    lp = h.lp(2, 3, [1, 2, 1])
    nb = C.c_size_t(0)
    assert h.lib.mipdhg_ipm_workspace_size(C.byref(lp), C.byref(nb)) == 0
    ws = h.buf(nb.value)
    words = np.ctypeslib.as_array(C.cast(ws, C.POINTER(C.c_int32)), (nb.value // 4,))
    assert h.ipm(lp, ws, nb.value) >= 0
    # the counters (replaced pivots, waits that ran out) start one of the workspace's slices, after the inverses: a
    # kernel that noted a wait there (kernels do not run here) is reported, a replaced pivot is no error
    found = []
    for at in range(0, nb.value // 4, 64):
        for word in (0, 1):
            words[:] = 0
            words[at + word] = 1
            if h.ipm(lp, ws, nb.value) == -4 and b"gave up waiting" in h.lib.mipdhg_last_error():
                found.append((at, word))
    assert len(found) == 1 and found[0][1] == 1, found
    """)
