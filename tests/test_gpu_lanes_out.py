"""GPU: batched results extracted straight into page-locked memory and through device rows:
around the vertex count at which the extraction's runs widen, odd row lengths (rows that begin
in the middle of a write), every row width, hub-sorted ids, and rows of both kinds in one
server batch, against the oracle's levels."""
import numpy as np
import pytest

import gen
import oracle
import paper_2208_14935_amd as hy

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hub", [False, True])
@pytest.mark.parametrize("n,lanes", [(65, 3), (1001, 37), (32767, 64), (32768, 5), (33001, 64)])
def test_pinned_rows_equal_pageable_rows(n, lanes, hub):
    off, col = gen.er(n, 4 * n, seed=7)
    srcs = np.random.default_rng(n).integers(0, n, lanes).astype(np.uint32)
    want = {int(s): oracle.bfs(off, col, int(s))[0] for s in np.unique(srcs)}
    with hy.Graph(off, col, hub_sort=hub) as g:
        pin = hy.pinned_empty(lanes * n + 9, np.uint32)
        pin[:] = 7
        page = np.full((lanes, n), 9, np.uint32)
        g.run_batch("bfs", srcs, out=pin[5:5 + lanes * n])
        g.run_batch("bfs", srcs, out=page)
    assert np.all(pin[:5] == 7) and np.all(pin[5 + lanes * n:] == 7)
    rows = pin[5:5 + lanes * n].reshape(lanes, n)
    for i, s in enumerate(srcs):
        assert np.array_equal(rows[i], want[int(s)]) and np.array_equal(page[i], want[int(s)])


def test_pinned_and_pageable_rows_of_one_server():
    n = 40_003
    off, col = gen.er(n, 4 * n, seed=9)
    srcs = np.random.default_rng(3).integers(0, n, 24).astype(np.uint32)
    with hy.Graph(off, col) as g, hy.Server(g, bfs=16, sssp=0, ppr=0) as srv:
        qs = [srv.submit("bfs", int(s), out=hy.pinned_empty(n, np.uint32) if i % 3 else np.empty(n, np.uint32))
              for i, s in enumerate(srcs)]
        for q in qs:
            srv.wait(q)
            assert np.array_equal(q.values, oracle.bfs(off, col, q.source)[0])
