"""GPU: components of graphs without a budget (joined in a parent forest) against the oracle:
graphs of many components, none of them large, chains in both orders (the deepest trees),
hubs outside the largest component, and vertices whose edges all lie beyond the sampled two."""
import numpy as np
import pytest

import gen
import oracle
import paper_2208_14935_amd as hy

pytestmark = pytest.mark.gpu


def both(n, u, v):
    u, v = np.asarray(u, np.uint32), np.asarray(v, np.uint32)
    return gen.from_pairs(n, np.concatenate([u, v]), np.concatenate([v, u]))


def chain(order):
    return both(len(order), order[:-1], order[1:])


def cliques(k, size):
    """k cliques of `size` vertices, interleaved: vertex v belongs to clique v mod k."""
    i, j = np.triu_indices(size, 1)
    u = (i[None, :] * k + np.arange(k)[:, None]).ravel()
    v = (j[None, :] * k + np.arange(k)[:, None]).ravel()
    return both(k * size, u, v)


def stars(n, hubs):
    """`hubs` hubs at the end of the ids, the other vertices dealt out to them."""
    u = np.arange(n - hubs)
    return both(n, u, n - 1 - u % hubs)


GRAPHS = {
    "2 vertices": lambda: both(2, [0], [1]),
    "no edges": lambda: (np.zeros(6, np.uint64), np.zeros(0, np.uint32)),
    "chain": lambda: chain(np.arange(20000)),
    "chain, shuffled ids": lambda: chain(np.random.default_rng(1).permutation(30011)),
    "cliques": lambda: cliques(700, 9),
    "two cliques": lambda: cliques(2, 130),
    "stars": lambda: stars(40000, 7),
    "sparse": lambda: gen.symmetrize(*gen.er(50001, 40000, seed=8)),
    "rmat": lambda: gen.symmetrize(*gen.rmat(14, 4, seed=14)),
}


@pytest.mark.parametrize("hub_sort", [False, True])
@pytest.mark.parametrize("name", list(GRAPHS))
def test_components_match_oracle(name, hub_sort):
    off, col = GRAPHS[name]()
    want = oracle.cc(off, col)[0]
    with hy.Graph(off, col, symmetric=True, hub_sort=hub_sort) as g:
        g.set_params(partition_edges=1024)
        res = g.run("cc", trace=True, stats=True)
        plain = g.run("cc")
    for r in (res, plain):
        np.testing.assert_array_equal(r.values, want)
        assert 1 <= r.iterations <= max(oracle.sync_rounds(off, col, None, "cc"), 1)
    if len(col):
        assert res.iters[0]["active_edges"] == len(col)
        if not hub_sort:  # partitions follow the held order
            edges = np.diff(off[oracle.partition(off, 1024).astype(np.int64)])
            assert (res.mode_trace[0][edges > 0] == hy.P_RESIDENT).all()
