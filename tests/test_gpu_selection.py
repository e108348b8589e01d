"""GPU: the selection kernels at their edges, against the oracle's engine choice: partitions of
many vertices (several 4,096-vertex units, more than the 64 that one pass of the combining
wave takes) and partition counts around the one-workgroup scan's 1,024, 4,096 and 16,384; and the one-launch selection
of graphs of at most 16 units."""
import numpy as np
import pytest

import gen
import oracle
import paper_2208_14935_amd as hy

pytestmark = pytest.mark.gpu


def bfs_trace(off, col, source, pe, distinct, resident):
    lvl, it = oracle.bfs(off, col, source)
    with hy.Graph(off, col) as g:
        g.set_params(partition_edges=pe, compact_chunk_edges=1 << 16, rq_distinct_lines=int(distinct))
        g.set_resident_fraction("bfs", resident)
        res = g.run("bfs", source, trace=True, stats=True)
        plain = g.run("bfs", source)
        bounds = g.partition_bounds()
        nres = res.stats["nres"]
    for r in (res, plain):
        assert np.array_equal(r.values, lvl) and r.iterations == it
    E = np.diff(off[bounds.astype(np.int64)])
    assert len(E) == res.stats["npart"]
    for t in range(it):
        nA, Ea, Rq = oracle.partition_stats(bounds, off, lvl == t, arrays=1, distinct=distinct)
        want = oracle.select(E, nA, Ea, Rq, nres=nres, params=oracle.CostParams())
        np.testing.assert_array_equal(res.mode_trace[t], want, err_msg=f"iteration {t}")
        assert res.iters[t]["active_edges"] == int(Ea.sum())
        assert res.iters[t]["active_vertices"] == int(nA.sum())
    return len(E)


@pytest.mark.parametrize("distinct", [False, True])
@pytest.mark.parametrize("pe", [3000, 1 << 17])
def test_partitions_of_many_units(pe, distinct):
    """700,001 vertices, most without out-edges: partitions of up to 170 units."""
    rng = np.random.default_rng(3)
    n = 700_001
    src = np.concatenate([np.zeros(4000, np.int64), rng.integers(0, n, 250_000)])
    dst = np.concatenate([rng.integers(0, n, 4000), rng.integers(0, n, 250_000)])
    off, col = gen.from_pairs(n, src.astype(np.uint32), dst.astype(np.uint32))
    bfs_trace(off, col, 0, pe, distinct, 0.25)


@pytest.mark.parametrize("npart", [1, 2, 1024, 1025, 4096, 4097, 16384, 16385])
def test_partition_counts_around_the_scan(npart):
    """Every vertex a partition of its own: vertex 0 leads to all others and they back."""
    n = max(npart, 2)
    spokes = np.arange(1, n, dtype=np.uint32)
    hub = np.zeros(n - 1, dtype=np.uint32)
    src, dst = np.concatenate([hub, spokes]), np.concatenate([spokes, hub])
    off, col = gen.from_pairs(n, src, dst)
    assert bfs_trace(off, col, n // 2, 1 if npart > 1 else 8, False, 0.5) == npart


def test_sssp_byte_weights_over_many_units():
    """The first two frontiers' engines with a byte weight array counted apart (d1 = 5)."""
    rng = np.random.default_rng(4)
    n = 300_000
    src = np.concatenate([np.zeros(30_000, np.int64), rng.integers(0, n, 200_000)])
    dst = np.concatenate([rng.integers(0, n, 30_000), rng.integers(0, n, 200_000)])
    off, col = gen.from_pairs(n, src.astype(np.uint32), dst.astype(np.uint32))
    w = gen.weights(off, col, 9)
    act = [np.zeros(n, bool), np.zeros(n, bool)]
    act[0][0] = act[1][col[off[0]:off[1]]] = True
    act[1][0] = False
    for distinct in (False, True):
        with hy.Graph(off, col, weights=w, pack=False) as g:
            g.set_params(partition_edges=1 << 16, compact_chunk_edges=1 << 16, rq_distinct_lines=int(distinct))
            g.set_resident_fraction("sssp", 0.2)
            res = g.run("sssp", 0, trace=True, stats=True)
            bounds = g.partition_bounds()
        assert np.array_equal(res.values, oracle.sssp(off, col, w, 0))
        E = np.diff(off[bounds.astype(np.int64)])
        for t in range(2):
            nA, Ea, Rq = oracle.partition_stats(bounds, off, act[t], arrays=2, weight_bytes=1, distinct=distinct)
            want = oracle.select(E, nA, Ea, Rq, nres=res.stats["nres"], params=oracle.CostParams(d1=5))
            np.testing.assert_array_equal(res.mode_trace[t], want, err_msg=f"iteration {t}")


@pytest.mark.parametrize("n", [65, 4096, 4097, 61440, 65536, 65537])
@pytest.mark.parametrize("pe", [1000, 1 << 20])
def test_small_graphs_around_the_one_launch_selection(n, pe):
    """Up to 16 units (of one partition, or of several) in one launch, 17 in four."""
    off, col = gen.er(n, 6 * n if n < 10_000 else n // 20, seed=n)
    source = int(np.nonzero(np.diff(off.astype(np.int64)))[0][0])
    for distinct in (False, True):
        bfs_trace(off, col, source, pe, distinct, 0.4)
    w = gen.weights(off, col, 5)
    srcs = np.nonzero(np.diff(off.astype(np.int64)))[0][:40].astype(np.uint32)
    with hy.Graph(off, col, weights=w) as g:
        assert np.array_equal(g.run("sssp", source).values, oracle.sssp(off, col, w, source))
        got, its, _ = g.run_batch("bfs", srcs)
        for l, s in enumerate(srcs):
            want, it = oracle.bfs(off, col, int(s))
            assert np.array_equal(got[l], want) and its[l] == it
