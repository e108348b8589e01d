"""GPU: PageRank over the gather plan (graphs without a budget): pairs sorted by destination
bin once, contributions gathered and summed in LDS every iteration, against the FP64 oracle.
Sizes lie around the bins' and wave groups' edges; the star puts more pairs into one bin
than a segment holds (its sums are joined by atomic adds); small pieces cut at any edge, so
pieces start in the middle of an eight-pair load."""
import numpy as np
import pytest

import gen
import oracle
import paper_2208_14935_amd as hy

pytestmark = pytest.mark.gpu


def star(n, m):
    """m edges from distinct vertices to vertex 0 and as many back, the rest isolated."""
    spokes = np.arange(1, m + 1, dtype=np.uint32)
    hub = np.zeros(m, dtype=np.uint32)
    return gen.from_pairs(n, np.concatenate([spokes, hub]), np.concatenate([hub, spokes]))


GRAPHS = {
    "one vertex": lambda: (np.zeros(2, np.uint64), np.zeros(0, np.uint32)),
    "65": lambda: gen.er(65, 300, seed=1),
    "4095": lambda: gen.er(4095, 20000, seed=2),
    "2^15 + 1": lambda: gen.er((1 << 15) + 1, 1 << 18, seed=3),
    "rmat 16": lambda: gen.rmat(16, 16, seed=16),
    "2^20 + 3": lambda: gen.er((1 << 20) + 3, 3 << 20, seed=4),
    "2^21 + 1": lambda: gen.er((1 << 21) + 1, 3 << 20, seed=5),  # 257 bins, the last of one vertex
    "2^23 + 1": lambda: gen.er((1 << 23) + 1, 9 << 20, seed=7),  # 1025 bins: two sorting passes
}


def check(res, want):
    got = res.values.astype(np.float64)
    # FP32 shares and sums of unequal terms, at most ~1e4 of them (R-MAT 16's largest in-degree)
    # in any order: 2^-24 = 6e-8 per rounding, growing as the square root of their number, 6e-6
    assert np.linalg.norm(got - want) <= 2e-5 * np.linalg.norm(want)
    assert np.abs(got - want).max() <= 1e-6
    assert res.iterations == 20


@pytest.mark.parametrize("pairs", [0, 5001])
@pytest.mark.parametrize("name", list(GRAPHS))
def test_plan_matches_oracle(name, pairs):
    off, col = GRAPHS[name]()
    if pairs and len(col) > 300 * pairs:
        pytest.skip("thousands of pieces")
    want = oracle.pagerank(off, col, 0.85, 20)
    with hy.Graph(off, col) as g:
        g.set_params(partition_edges=2048, pr_block_pairs=pairs)
        first = g.run("pagerank")
        check(first, want)
        check(g.run("pagerank"), want)  # over the kept plan


def test_bin_of_several_segments():
    """50000 pairs of one destination (segments hold 16384).  With 2^16 vertices the first
    step's shares are 2^-16 and their sums exact in FP32, so a lost or doubled pair shows."""
    off, col = star(1 << 16, 50000)
    want = oracle.pagerank(off, col, 0.85, 1)
    with hy.Graph(off, col) as g:
        g.set_params(pr_iterations=1)
        for _ in range(2):
            got = g.run("pagerank").values
            assert np.abs(got / want - 1).max() <= 1e-6  # a few roundings; a pair is 2e-5 of the hub's sum


def test_plan_follows_budget_pieces_and_steps():
    """The plan is remade for other piece sizes and given up for a budget; a run of another
    number of steps, and one that does not block, go with it."""
    off, col = gen.rmat(14, 16, seed=14)
    want = oracle.pagerank(off, col, 0.85, 20)
    with hy.Graph(off, col, weights=gen.weights(off, col, 3)) as g:  # packed edge words
        g.set_params(partition_edges=2048)
        check(g.run("pagerank"), want)
        g.set_params(pr_block_pairs=9999)
        check(g.run("pagerank"), want)
        g.set_params(partition_edges=4096)
        check(g.run("pagerank"), want)
        g.set_resident_fraction("pagerank", 0.5)
        check(g.run("pagerank"), want)
        g.set_budget(None)
        check(g.run("pagerank"), want)
        assert np.array_equal(g.run("bfs", 1).values, oracle.bfs(off, col, 1)[0])
        check(g.run("pagerank"), want)
        g.set_params(pr_iterations=1)
        one = g.run("pagerank").values
        assert np.abs(one - oracle.pagerank(off, col, 0.85, 1)).max() <= 1e-6
        g.set_params(pr_blocking=0, pr_iterations=20)
        check(g.run("pagerank"), want)


@pytest.mark.parametrize("hub_sort", [False, True])
def test_plan_on_a_union_of_graphs(hub_sort):
    graphs = [gen.rmat(10, 8, seed=1), gen.er(777, 5000, seed=2), gen.rmat(12, 8, seed=3)]
    off, col, _, bounds = gen.disjoint_union(graphs)
    with hy.Graph(off, col, hub_sort=hub_sort) as g:
        g.set_parts(bounds)
        got = g.run("pagerank").values
    for i, (o, c) in enumerate(graphs):
        want = oracle.pagerank(o, c, 0.85, 20)
        assert np.abs(got[int(bounds[i]):int(bounds[i + 1])] - want).max() <= 1e-6


@pytest.mark.parametrize("mode", ["hybrid", "filter", "zerocopy"])
@pytest.mark.parametrize("resident", [0.05, 0.3, 0.7])
@pytest.mark.parametrize("name", ["4095", "2^15 + 1", "rmat 16", "2^20 + 3", "2^21 + 1"])
def test_compact_plan_matches_oracle(name, resident, mode):
    """Budgeted graphs: the resident edges in one-word pairs, sources in blocks of 2^16."""
    off, col = GRAPHS[name]()
    want = oracle.pagerank(off, col, 0.85, 20)
    with hy.Graph(off, col) as g:
        g.set_params(partition_edges=512, mode=mode, compact_chunk_edges=1 << 14)
        g.set_resident_fraction("pagerank", resident)
        first = g.run("pagerank", stats=True)
        check(first, want)
        check(g.run("pagerank"), want)
        assert 0 < first.stats["nres"] < first.stats["npart"]
        g.set_params(pr_blocking=0)
        off_run = g.run("pagerank", stats=True)
        check(off_run, want)
        # the same partitions are read over the link: only the resident adds changed
        assert first.stats["active_edges"] == off_run.stats["active_edges"]
        assert first.stats["nres"] == off_run.stats["nres"]


def test_compact_plan_ends_inside_the_resident_prefix():
    """More resident edges than 16 MiB hold pairs for (2^20 vertices, 6.3M resident edges): the
    partitions past the plan's are added atomically."""
    rng = np.random.default_rng(2)
    n = 1 << 20
    off, col = gen.from_pairs(n, rng.integers(0, n // 8, 9 << 20).astype(np.uint32),
                              rng.integers(0, n, 9 << 20).astype(np.uint32))
    want = oracle.pagerank(off, col, 0.85, 20)
    with hy.Graph(off, col) as g:
        g.set_resident_fraction("pagerank", 0.7)
        res = g.run("pagerank", stats=True, time_kernels=True)
        check(res, want)
        check(g.run("pagerank"), want)
        g.set_resident_fraction("pagerank", 0.2)  # another plan
        check(g.run("pagerank"), want)
    assert res.stats["kernel_launches"][hy.KERNEL_CLASSES.index("push_resident")] >= 20  # the rest of them
    assert res.stats["kernel_launches"][hy.KERNEL_CLASSES.index("pr_blocking")] == 20


def test_compact_plan_of_many_bins():
    """17M vertices: 4,151 bins of 2^12 vertices."""
    off, col = gen.er(17_000_000, 34_000_000, seed=9)
    want = oracle.pagerank(off, col, 0.85, 20)
    with hy.Graph(off, col) as g:
        g.set_resident_fraction("pagerank", 0.4)
        check(g.run("pagerank"), want)


def test_compact_plan_of_wide_bins():
    """2^25 + 1 vertices: bins of 2^12 would be one more than the 8,192 that the sort counts in LDS, so
    they hold 2^13.  Two iterations: at most ~10 equal shares per sum, each rounded to FP32."""
    off, col = gen.er((1 << 25) + 1, 34_000_000, seed=9)
    want = oracle.pagerank(off, col, 0.85, 2)
    with hy.Graph(off, col) as g:
        g.set_params(pr_iterations=2)
        g.set_resident_fraction("pagerank", 0.3)
        for _ in range(2):
            got = g.run("pagerank").values.astype(np.float64)
            assert np.linalg.norm(got - want) <= 2e-6 * np.linalg.norm(want)


def test_pieces_are_run_where_they_are_asked_for():
    """pr_blocking = 2 sorts each piece anew in every iteration, also over a fully resident graph:
    preparing and applying are launches of their own there, one pass over the kept plan."""
    off, col = GRAPHS["rmat 16"]()
    want = oracle.pagerank(off, col, 0.85, 20)
    other, block = hy.KERNEL_CLASSES.index("other"), hy.KERNEL_CLASSES.index("pr_blocking")
    with hy.Graph(off, col) as g:
        g.set_params(pr_block_pairs=200_000)
        for blocking in (1, 2):
            g.set_params(pr_blocking=blocking)
            g.run("pagerank")
            res = g.run("pagerank", time_kernels=True)
            check(res, want)
            assert res.stats["kernel_launches"][block] >= 20 * 4
            assert (res.stats["kernel_launches"][other] >= 40) == (blocking == 2)


@pytest.mark.parametrize("degree,planned", [(3, True), (12, False)])
def test_plan_or_pieces_by_the_share_that_the_plan_covers(degree, planned):
    """More than 3/8 resident: 16 bytes per vertex hold the pairs of every resident edge (2.1 per
    vertex), which take one launch an iteration; or of half of them (8.4), which go in pieces."""
    n = (1 << 20) + 3
    off, col = gen.er(n, degree * n, seed=6)
    want = oracle.pagerank(off, col, 0.85, 20)
    with hy.Graph(off, col) as g:
        g.set_params(pr_block_pairs=1 << 20)
        g.set_resident_fraction("pagerank", 0.7)
        res = g.run("pagerank", time_kernels=True)
        check(res, want)
        launches = res.stats["kernel_launches"][hy.KERNEL_CLASSES.index("pr_blocking")]
        assert launches == 20 if planned else launches >= 20 * 8


def test_plan_of_widest_bins():
    """2^27 + 1 vertices: bins of 2^13 would be one more than the sort's 2^14, so they hold 2^14 sums.
    Two iterations of few equal shares, each rounded to FP32; the second over the kept plan's pairs."""
    off, col = gen.er((1 << 27) + 1, 2_000_000, seed=10)
    want = oracle.pagerank(off, col, 0.85, 2)
    with hy.Graph(off, col) as g:
        g.set_params(pr_iterations=2)
        for _ in range(2):
            got = g.run("pagerank").values
            assert np.abs(got / want - 1).max() <= 2e-6
