"""Queries in arenas that hold their largest level and little else: what the
fused kernels use is given back before the per-level kernels run, and so is
what a join turned out too small for its level was launched with."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is loaded before the library)

import workloads as w

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def graph():
    r = np.random.default_rng(4)
    n, m = 30_000, 600_000
    a, b = r.integers(0, n, int(1.1 * m) + 16), r.integers(0, n, int(1.1 * m) + 16)
    keys = r.permutation(np.unique(np.minimum(a, b)[a != b].astype(np.int64) << 32 | np.maximum(a, b)[a != b]))[:m]
    return w.make_graph(n, r.integers(0, 3, n), np.stack([keys >> 32, keys & 0xFFFFFFFF], 1), r.integers(0, 1, m), "r")


# levels of 2.4 * 10^7 rows, 385 MB of result, and of 3 * 10^8 rows, 6.1 GB
@pytest.mark.parametrize("k,count_only,kib", [(4, True, 113_950), (4, False, 463_600), (5, False, 7_153_500)])
def test_largest_level_fits(graph, k, count_only, kib):
    import paper_1906_03420_amd as gsi
    q = w.QueryMaker(graph).make(k, "walk", 100 + k)
    flags = gsi.GSI_COUNT_ONLY if count_only else gsi.GSI_NO_CHUNKS
    print(k, count_only, kib, flush=True)
    with gsi.Context(kib << 10) as ctx:
        dg = ctx.load(graph)
        r = dg.query(q, flags=flags)
        count, digest = r.count, r.digest
        r.free()
        r = dg.query(q, flags=gsi.GSI_COUNT_ONLY | gsi.GSI_NO_FUSED)
        assert (count, digest) == (r.count, r.digest)
        r.free()
        dg.free()


def test_level_joined_twice_fits():
    """1,024 roots with 470 leaves each where 64 slots a row are expected: the
    join sized for 65,536 slots leaves the room of its records to the one that
    takes all 481,280.  Kept results XX."""
    import paper_1906_03420_amd as gsi
    roots, fan, free = 1024, 470, 4_500_000
    a = np.repeat(np.arange(roots), fan)
    b = roots + np.arange(roots * fan)
    g = w.make_graph(roots + roots * fan, np.repeat([0, 1], [roots, roots * fan]), np.stack([a, b], 1),
                     [0] * len(a), "fans")
    pair = w.make_query([0, 1], [(0, 1)], [0])
    size = gsi.gsi_graph_bytes_needed(g.n, g.m)
    with gsi.Context(size) as ctx:
        dg = ctx.load(g)
        kept = []
        for lab, rows in ((1, roots * fan), (0, roots)):
            q = w.make_query([lab], [], [])
            while size - ctx.memory()[0] - 4 * rows >= free:
                kept.append(dg.query(q))
                assert kept[-1].count == rows
        r = dg.query(pair, flags=gsi.GSI_NO_FUSED, order=[0, 1])
        assert r.stats()["gba"][1] == len(a)
        np.testing.assert_array_equal(r.rows(), np.stack([a, b], 1))
        r.free()
        for r in kept:
            r.free()
        dg.free()
