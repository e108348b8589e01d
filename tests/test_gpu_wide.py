"""GPU: iterations whose improved vertices are reported by plain stores (from n/32 active edges
on), against the oracle: iteration counts and values with partitions that begin inside a
64-vertex window, odd vertex counts, frontiers on both sides of the rule in one run, and runs
of more such iterations than the marks have tags."""
import numpy as np
import pytest

import gen
import oracle
import paper_2208_14935_amd as hy

pytestmark = pytest.mark.gpu


def layers(count, width, back):
    """`count` layers of `width` vertices: every vertex leads to the whole next layer and to
    `back` random vertices of earlier layers."""
    rng = np.random.default_rng(5)
    src, dst = [], []
    for k in range(count):
        ids = np.arange(k * width, (k + 1) * width)
        if k + 1 < count:
            src.append(np.repeat(ids, width))
            dst.append(np.tile(ids + width, width))
        if k:
            src.append(np.repeat(ids, back))
            dst.append(rng.integers(0, k * width, width * back))
    n = count * width
    key = np.unique(np.concatenate(src).astype(np.int64) * n + np.concatenate(dst))
    off = np.searchsorted(key, np.arange(n + 1) * n).astype(np.uint64)
    return off, (key % n).astype(np.uint32)


@pytest.mark.parametrize("resident", [1.0, 0.3])
def test_more_wide_iterations_than_tags(resident):
    # every frontier is one layer: about 4 * 24 edges, above 1200 / 32
    off, col = layers(300, 4, 20)
    w = np.full(len(col), 3, np.uint32)
    with hy.Graph(off, col, weights=w) as g:
        for algo in ("bfs", "sssp"):
            g.set_params(partition_edges=512)
            g.set_resident_fraction(algo, resident)
            for _ in range(2):
                r = g.run(algo, 0)
                lvl, it = oracle.bfs(off, col, 0)
                assert np.array_equal(r.values, lvl if algo == "bfs" else lvl * 3)
                assert algo != "bfs" or r.iterations == it
    assert it > 256


@pytest.mark.parametrize("resident", [1.0, 0.4])
@pytest.mark.parametrize("n,m,pe", [(70_001, 900_000, 777), (262_143, 700_000, 1 << 15), (131_073, 2_000_000, 100)])
def test_wide_and_narrow_iterations(n, m, pe, resident):
    off, col = gen.er(n, m, seed=n)
    w = np.random.default_rng(n).integers(1, 65, len(col)).astype(np.uint32)
    s = int(gen.sources(off, 1, 3)[0])
    with hy.Graph(off, col, weights=w) as g:
        g.set_params(partition_edges=pe)
        for algo in ("bfs", "sssp"):
            g.set_resident_fraction(algo, resident)
            for _ in range(2):
                r = g.run(algo, s)
                if algo == "bfs":
                    lvl, it = oracle.bfs(off, col, s)
                    assert np.array_equal(r.values, lvl) and r.iterations == it
                else:
                    assert np.array_equal(r.values, oracle.sssp(off, col, w, s))


@pytest.mark.parametrize("n,m,pe", [(70_001, 200_000, 777), (131_073, 400_000, 1 << 14)])
def test_wide_components(n, m, pe):
    off, col = gen.er(n, m, seed=n)
    soff, scol = gen.symmetrize(off, col)
    with hy.Graph(soff, scol, symmetric=True) as g:
        g.set_params(partition_edges=pe)
        g.set_resident_fraction("cc", 0.4)
        r = g.run("cc")
    assert np.array_equal(r.values, oracle.cc(soff, scol)[0])


@pytest.mark.parametrize("resident", [1.0, 0.3])
@pytest.mark.parametrize("lanes", [1, 2, 7, 33, 64])
def test_wide_batches(lanes, resident):
    n = 70_001
    off, col = gen.er(n, 500_000, seed=4)
    srcs = gen.sources(off, lanes, 11)
    with hy.Graph(off, col) as g:
        g.set_params(partition_edges=1000)
        g.set_resident_fraction("bfs", resident)
        vals, its, _ = g.run_batch("bfs", srcs)
        with hy.Server(g, bfs=8, sssp=0, ppr=0) as srv:  # lanes that join at different iterations
            qs = [srv.submit("bfs", int(s)) for s in srcs]
            for q in qs:
                srv.wait(q)
    for i, s in enumerate(srcs):
        lvl, it = oracle.bfs(off, col, int(s))
        assert np.array_equal(vals[i], lvl) and its[i] == it
        assert np.array_equal(qs[i].values, lvl) and qs[i].result["iterations"] == it
