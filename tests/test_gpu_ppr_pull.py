"""GPU: personalized PageRank and batched SSSP steps over the in-edge lists (dense steps of
graphs without a budget) against the oracle (PPR in FP64, distances exact): row widths from 1 to
64 lanes, edge counts around the runs' 64 (rows of up to 32 lanes) and 128 edges (64 lanes) of
small graphs, the 256 of large ones and a segment's 256, and in-lists spanning many runs and
segments."""
import numpy as np
import pytest

import gen
import oracle
import paper_2208_14935_amd as hy

pytestmark = pytest.mark.gpu


def star(n, m):
    spokes = np.arange(1, m + 1, dtype=np.uint32)
    hub = np.zeros(m, dtype=np.uint32)
    return gen.from_pairs(n, np.concatenate([spokes, hub]), np.concatenate([hub, spokes]))


def ring(n):
    """n vertices of one in- and one out-edge, and an isolated one."""
    v = np.arange(n, dtype=np.uint32)
    return gen.from_pairs(n + 1, v, (v + 1) % n)


GRAPHS = {
    "2 edges": lambda: ring(2),
    "63 edges": lambda: ring(63),
    "64 edges": lambda: ring(64),
    "65 edges": lambda: ring(65),
    "127 edges": lambda: ring(127),
    "128 edges": lambda: ring(128),
    "129 edges": lambda: ring(129),
    "star": lambda: star(3000, 2500),
    "er": lambda: gen.er(1001, 9000, seed=5),
    "rmat": lambda: gen.rmat(11, 16, seed=11),
}


@pytest.mark.parametrize("lanes", [1, 2, 3, 8, 9, 17, 33, 64])
@pytest.mark.parametrize("name", list(GRAPHS))
def test_pulled_steps_match_oracle(name, lanes):
    off, col = GRAPHS[name]()
    rng = np.random.default_rng(lanes)
    srcs = rng.choice(np.nonzero(np.diff(off.astype(np.int64)))[0], lanes).astype(np.uint32)
    srcs[-1] = srcs[0]  # a repeated source
    with hy.Graph(off, col) as g:
        got, iters, _ = g.run_batch("ppr", srcs)
        again, _, _ = g.run_batch("ppr", srcs)
    assert (iters == 10).all()
    for l, s in enumerate(srcs):
        want = oracle.ppr(off, col, int(s), 0.85, 10)
        for x in (got[l], again[l]):
            # per step one FP32 rounding of the share and one of the value, sums in FP64: ten
            # steps keep every value within 20 * 2^-24 = 1.2e-6 of itself
            assert np.all(np.abs(x - want) <= 1.3e-6 * want + 1e-30)


def test_in_lists_are_given_up_for_a_budget():
    off, col = gen.rmat(12, 16, seed=12)
    with hy.Graph(off, col) as g:
        g.set_params(partition_edges=2048, compact_chunk_edges=4096)
        want = oracle.ppr(off, col, 7, 0.85, 10)
        for budget in (False, True, False):
            if budget:
                g.set_resident_fraction("ppr", 0.4)
            else:
                g.set_budget(None)
            assert np.abs(g.run("ppr", 7).values - want).max() <= 1e-6


@pytest.mark.parametrize("lanes", [8, 9, 17, 64])
@pytest.mark.parametrize("weights", ["packed", "bytes", "words"])
@pytest.mark.parametrize("name", list(GRAPHS))
def test_pulled_sssp_matches_oracle(name, weights, lanes):
    off, col = GRAPHS[name]()
    w = gen.weights(off, col, 77)
    rng = np.random.default_rng(lanes)
    srcs = rng.choice(np.nonzero(np.diff(off.astype(np.int64)))[0], lanes).astype(np.uint32)
    with hy.Graph(off, col, weights=w, pack=weights == "packed", narrow=weights != "words") as g:
        g.run_batch("ppr", srcs)  # lists without weights come first
        got, _, _ = g.run_batch("sssp", srcs)
        again, _, _ = g.run_batch("sssp", srcs)
    for s in set(srcs.tolist()):
        want = oracle.sssp(off, col, w, s)
        for l in np.nonzero(srcs == s)[0]:
            assert np.array_equal(got[l], want) and np.array_equal(again[l], want)


def test_pulled_sssp_reports_overflow():
    """One lane's distances pass 2^32 - 1 over a dense step, the others' do not exist."""
    n = 40
    v = np.arange(n - 1, dtype=np.uint32)
    off, col = gen.from_pairs(n, v, v + 1)
    w = np.full(len(col), 0x20000000, dtype=np.uint32)
    srcs = np.arange(20, 40, dtype=np.uint32)
    with hy.Graph(off, col, weights=w) as g:
        with pytest.raises(hy.HytmError) as ei:
            g.run_batch("sssp", srcs)
        assert ei.value.status == hy.E_RANGE
        got, _, _ = g.run_batch("sssp", srcs[13:].repeat(3))  # at most six edges from the end
        for l, s in enumerate(srcs[13:].repeat(3)):
            assert np.array_equal(got[l], oracle.sssp(off, col, w, int(s)))


def test_pulled_runs_of_a_large_graph():
    """Rows of 64 lanes over 3.4M edges, which go in runs of 256: lists of about 110 edges, cut by
    the runs anywhere, and one of 20000 that spans many."""
    n, hub = 30_000, np.arange(1, 20_001, dtype=np.uint32)
    rng = np.random.default_rng(9)
    src = np.concatenate([rng.integers(0, n, 3_400_000).astype(np.uint32), hub])
    dst = np.concatenate([rng.integers(0, n, 3_400_000).astype(np.uint32), np.zeros(len(hub), np.uint32)])
    off, col = gen.from_pairs(n, src, dst)
    assert len(col) >= 256 * 12288
    w = gen.weights(off, col, 4)
    srcs = rng.choice(n, 4).astype(np.uint32)
    with hy.Graph(off, col, weights=w) as g:
        ppr, _, _ = g.run_batch("ppr", np.tile(srcs, 16))
        dist, _, _ = g.run_batch("sssp", np.tile(srcs, 16))
    for k, s in enumerate(srcs):
        want, wd = oracle.ppr(off, col, int(s), 0.85, 10), oracle.sssp(off, col, w, int(s))
        for l in range(k, 64, 4):
            # as above, and the FP64 sums' own roundings are far below
            assert np.all(np.abs(ppr[l] - want) <= 1.3e-6 * want + 1e-30)
            assert np.array_equal(dist[l], wd)


@pytest.mark.parametrize("lanes", [1, 2, 4, 12, 33, 64])
@pytest.mark.parametrize("n", [61, 5003, (1 << 20) + 3])
def test_sparse_steps_match_oracle(n, lanes):
    """One edge a vertex: few cells are active, in windows of a few rows (small graphs) to 64 vertices
    (from 2^20), the last one cut off."""
    off, col = gen.er(n, n, seed=n)
    rng = np.random.default_rng(lanes)
    srcs = rng.choice(np.nonzero(np.diff(off.astype(np.int64)))[0], min(lanes, 3)).astype(np.uint32)
    with hy.Graph(off, col) as g:
        got, _, _ = g.run_batch("ppr", np.resize(srcs, lanes))
    for k, s in enumerate(srcs):
        want = oracle.ppr(off, col, int(s), 0.85, 10)
        for l in range(k, lanes, len(srcs)):
            assert np.all(np.abs(got[l] - want) <= 1.3e-6 * want + 1e-30)  # as above
