"""GPU: the sorted forms of the edges that a graph keeps between calls (PageRank's plans, the
in-edge lists) are caches.  Without room for them, or with a limit of none, calls go without
and give the oracle's results; a call that finds the device full has them given back, also by
other handles.  A full device is one whose remaining room this thread's calls are told
(hytm_test_device_room), so nothing is filled."""
import contextlib
import ctypes
import threading

import numpy as np
import pytest

import gen
import oracle
import paper_2208_14935_amd as hy

pytestmark = pytest.mark.gpu

RES, OTHER, BLOCK = (hy.KERNEL_CLASSES.index(c) for c in ("push_resident", "other", "pr_blocking"))
N, SCALE = 1 << 16, 16


@contextlib.contextmanager
def room(nbytes):
    f = hy.load().hytm_test_device_room
    f.argtypes, f.restype = [ctypes.c_uint64], None
    f(int(nbytes))
    try:
        yield
    finally:
        f(hy.UNCAPPED)


@pytest.fixture(scope="module")
def rmat():
    off, col = gen.rmat(SCALE, 16, seed=SCALE)
    w = gen.weights(off, col, 3)
    want = {"pagerank": oracle.pagerank(off, col, 0.85, 20), "ppr": oracle.ppr(off, col, 7, 0.85, 10),
            "sssp": oracle.sssp(off, col, w, 7), "bfs": oracle.bfs(off, col, 7)[0]}
    return off, col, w, want


def check_pagerank(res, want):
    # FP32 shares and sums of at most ~1e4 unequal terms in any order: 6e-6 (6e-8 times the
    # square root of their number)
    got = res.values.astype(np.float64)
    assert np.linalg.norm(got - want) <= 2e-5 * np.linalg.norm(want)


def other_launches(g, algo, lanes=0):
    if lanes:
        return g.run_batch(algo, [7] * lanes, time_kernels=True)[2]["kernel_launches"][OTHER]
    return g.run(algo, 7, time_kernels=True).stats["kernel_launches"][OTHER]


@pytest.mark.parametrize("how", ["limit", "room"])
def test_calls_go_without_plans(rmat, how):
    off, col, w, want = rmat
    with hy.Graph(off, col, weights=w) as g:
        # everything but the plans is in place; then there is no room for them
        for algo in ("pagerank", "pagerank_delta", "ppr", "sssp"):
            g.run(algo, 7)
        g.run_batch("sssp", [7] * 20)
        g.set_plan_limit(0)
        g.run("pagerank")  # the pieces' buffers
        planned = other_launches(g, "pagerank")
        assert planned >= 41  # an initialisation, and preparing and applying in 20 iterations
        if how == "room":
            g.set_plan_limit(None)
        with room(1 << 20) if how == "room" else contextlib.nullcontext():
            for _ in range(2):
                res = g.run("pagerank", time_kernels=True)
                check_pagerank(res, want["pagerank"])
                assert res.stats["kernel_launches"][OTHER] == planned
                assert res.stats["kernel_launches"][BLOCK] >= 20
                assert np.abs(g.run("ppr", 7).values - want["ppr"]).max() <= 1e-6
                assert np.array_equal(g.run_batch("sssp", [7] * 20)[0][19], want["sssp"])
            pushed = other_launches(g, "ppr")
        g.set_plan_limit(None)
        check_pagerank(g.run("pagerank"), want["pagerank"])
        assert other_launches(g, "pagerank") < planned  # the plan is made and used again
        assert other_launches(g, "ppr") == pushed + 1   # the lists are made
        assert other_launches(g, "ppr") == pushed


@pytest.mark.parametrize("blocked", [False, True])
def test_budgeted_pagerank_goes_without_its_plan(rmat, blocked):
    """A quarter resident: atomic adds; more than 3/8: the pieces."""
    off, col, _, want = rmat
    with hy.Graph(off, col) as g:
        g.set_params(partition_edges=2048, compact_chunk_edges=1 << 14)
        g.set_resident_fraction("pagerank", 0.6 if blocked else 0.2)
        with_plan = g.run("pagerank", time_kernels=True)
        g.set_plan_limit(0)
        without = g.run("pagerank", time_kernels=True)
        for r in (with_plan, without):
            check_pagerank(r, want["pagerank"])
        assert (without.stats["kernel_launches"][BLOCK] > 0) == blocked
        g.set_plan_limit(None)
        with room(1 << 18):
            check_pagerank(g.run("pagerank"), want["pagerank"])
        check_pagerank(g.run("pagerank"), want["pagerank"])


def test_plans_make_way_for_a_call_of_the_same_graph(rmat):
    """8 PPR lanes need 7.3 MB of 4 MB; PageRank's plan (6 MB) and the lists (9 MB) are kept."""
    off, col, w, want = rmat
    with hy.Graph(off, col, weights=w) as g:
        for algo in ("pagerank", "ppr"):
            g.run(algo, 7)
        out = hy.pinned_empty((8, N), np.float32)
        with room(4 << 20):
            got, _, _ = g.run_batch("ppr", [7] * 8, out=out)
        for row in got:
            assert np.abs(row - want["ppr"]).max() <= 1e-6
        check_pagerank(g.run("pagerank"), want["pagerank"])


def test_plans_make_way_for_another_graph(rmat):
    off, col, w, want = rmat
    with hy.Graph(off, col) as a:
        check_pagerank(a.run("pagerank"), want["pagerank"])  # keeps 6 MB
        with room(2 << 20):
            with hy.Graph(off, col) as b:
                assert np.array_equal(b.run("bfs", 7).values, want["bfs"])  # 4 MB of edges
        check_pagerank(a.run("pagerank"), want["pagerank"])


def test_a_full_device_without_plans_is_reported(rmat):
    off, col, w, want = rmat
    with hy.Graph(off, col) as g:
        with room(1 << 20):
            with pytest.raises(hy.HytmError) as ei:
                g.run("bfs", 7)
        assert ei.value.status == hy.E_NOMEM
        assert np.array_equal(g.run("bfs", 7).values, want["bfs"])


def test_lists_of_an_open_server_stay(rmat):
    off, col, w, want = rmat
    with hy.Graph(off, col) as a:
        with hy.Server(a, bfs=0, sssp=0, ppr=2) as srv:
            assert np.abs(srv.wait(srv.submit("ppr", 7)).values - want["ppr"]).max() <= 1e-6
            with room(1 << 20):
                with pytest.raises(hy.HytmError) as ei:
                    with hy.Graph(off, col) as b:
                        b.run("bfs", 7)
            assert ei.value.status == hy.E_NOMEM
            assert np.abs(srv.wait(srv.submit("ppr", 7)).values - want["ppr"]).max() <= 1e-6


@pytest.mark.parametrize("spare", [0, 1 << 30])
def test_server_lists_stay_within_the_state_budget(rmat, spare):
    off, col, w, want = rmat
    with hy.Graph(off, col) as g:
        need = N * 8 * 4 + hy.Server.state_bytes(g, "ppr", 3)
        with hy.Server(g, bfs=0, sssp=0, ppr=3, state_budget=need + spare) as srv:
            for t in [srv.submit("ppr", 7) for _ in range(5)]:
                assert np.abs(srv.wait(t).values - want["ppr"]).max() <= 1e-6
        # lists that the server made are there for later calls, those it did not are made now
        first, second = other_launches(g, "ppr"), other_launches(g, "ppr")
        assert first == second + (0 if spare else 1)


def test_wide_iterations_without_marks(rmat):
    """One byte per vertex for wide SSSP iterations; without it the run goes on without them."""
    off, col, w, want = rmat
    with hy.Graph(off, col, weights=w) as g:
        g.set_params(sssp_delta=8)
        g.run("sssp", 7)  # every buffer but the marks
        g.set_params(sssp_delta=0)
        with room(N - 1):
            assert np.array_equal(g.run("sssp", 7).values, want["sssp"])
        assert np.array_equal(g.run("sssp", 7).values, want["sssp"])


def test_plans_are_taken_while_their_graph_is_called_from_another_thread(rmat):
    off, col, w, want = rmat
    errors = []

    def ranks(g):
        try:
            for _ in range(20):
                check_pagerank(g.run("pagerank"), want["pagerank"])
        except BaseException as e:  # noqa: BLE001 - reported by the test's thread
            errors.append(e)

    with hy.Graph(off, col) as a, hy.Graph(off, col) as b:
        t = threading.Thread(target=ranks, args=(a,))
        t.start()
        while t.is_alive():
            b.set_budget(1 << 20)  # lets the edges' room go
            b.run("bfs", 7)
            b.set_budget(None)
            with room(2 << 20):
                try:
                    assert np.array_equal(b.run("bfs", 7).values, want["bfs"])
                except hy.HytmError as e:  # a's plan was in use or not there
                    assert e.status == hy.E_NOMEM
        t.join()
    assert not errors, errors
