"""The level-synchronous engine against the single-query path: survivor
records and, in an arena too small for them, keep bits; every group width;
workgroups whose survivors are of several queries; counts only and rows."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is loaded before the library)

import workloads as w

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def world():
    """A graph, queries of one to thousands of embeddings, and their answers."""
    import paper_1906_03420_amd as gsi
    r = np.random.default_rng(3)
    n = 600
    e = sorted({tuple(sorted(x)) for x in r.integers(0, n, (12000, 2)).tolist() if x[0] != x[1]})
    g = w.make_graph(n, r.integers(0, 3, n), e, r.integers(0, 2, len(e)), "engine")
    mk = w.QueryMaker(g)
    qs = [mk.make(2 + i % 4, ("walk", "tree", "dense")[i % 3], 100 + i) for i in range(40)]
    with gsi.Context(1 << 30) as ctx:
        dg = ctx.load(g)
        want = []
        for q in qs:
            res = dg.query(q)
            want.append((res.count, res.digest, res.sorted_rows()))
            res.free()
        dg.free()
    return g, qs, want


@pytest.mark.parametrize("arena_mib,bits", [(1024, False), (12, True)])
@pytest.mark.parametrize("tiles", [1, 2, 4, 8])
@pytest.mark.parametrize("count_only", [False, True])
def test_engine_matches_single_queries(world, arena_mib, bits, tiles, count_only):
    import paper_1906_03420_amd as gsi
    g, qs, want = world
    flags = gsi.GSI_BATCH_LEVELS_ONLY | (gsi.GSI_COUNT_ONLY if count_only else 0)
    print(arena_mib, tiles, count_only, flush=True)
    with gsi.Context(arena_mib << 20, flags=gsi.GSI_CTX_PROFILE) as ctx:
        dg = ctx.load(g)
        ctx.kernel_stats_reset()
        # the small arena holds one query's rows and steps at a time
        for part in ([qs] if not bits else [[q] for q in qs]):
            b = dg.batch(part, flags=flags, engine_tiles=tiles, threads=256, grid_scale=8)
            counts, digests = b.results()
            for i, q in enumerate(part):
                n, dig, rows = want[next(t for t, x in enumerate(qs) if x is q)]
                assert int(counts[i]) == n and tuple(int(x) for x in digests[i]) == dig
                if not count_only:
                    np.testing.assert_array_equal(b.sorted_rows(i), rows)
            b.free()
        ran = {k["name"]: k["launches"] for k in ctx.kernel_stats()}
        assert ran.get("k_wlink", 0) > 0
        assert (ran.get("k_wlink_bits", 0) > 0) == bits
        dg.free()


@pytest.mark.parametrize("n,k", [(40, 5), (47, 5)])
def test_engine_filtered_lists(n, k):
    """Rows that rescan a complete graph's few lists: the step filters the
    lists of the queries that would save 2^24 slots, beside one that would
    not; closed forms (falling factorials per label) and the single path."""
    import paper_1906_03420_amd as gsi
    g = w.complete_graph(n)
    g.vlabel[:] = np.arange(n) % 2
    na, nb = (n + 1) // 2, n // 2
    path = [(i, i + 1) for i in range(k - 1)]
    qs = [w.make_query([0] * k, path, [0] * (k - 1)),
          w.make_query([i % 2 for i in range(k)], path, [0] * (k - 1)),
          w.make_query([1] * k, path + [(0, k - 1)], [0] * k),
          w.make_query([0, 1], [(0, 1)], [0])]
    ff = lambda x, t: int(np.prod([x - i for i in range(t)], dtype=np.int64))  # noqa: E731
    want = [ff(na, k), ff(na, (k + 1) // 2) * ff(nb, k // 2), ff(nb, k), na * nb]
    reps = 8  # of the first query: its last levels alone pass 2^24 slots
    with gsi.Context(8 << 30, flags=gsi.GSI_CTX_PROFILE) as ctx:
        dg = ctx.load(g)
        single = []
        for q in qs:
            r = dg.query(q, flags=gsi.GSI_COUNT_ONLY)
            single.append(r.digest)
            r.free()
        ctx.kernel_stats_reset()
        b = dg.batch(qs + qs[:1] * (reps - 1), flags=gsi.GSI_COUNT_ONLY | gsi.GSI_BATCH_LEVELS_ONLY)
        counts, digests = b.results()
        b.free()
        for i, c in enumerate(counts.tolist()):
            j = i if i < len(qs) else 0
            assert c == want[j] and tuple(int(x) for x in digests[i]) == single[j]
        ran = {x["name"]: x["launches"] for x in ctx.kernel_stats()}
        assert ran.get("k_fn_bits", 0) > 0 and ran.get("k_fn_relocate", 0) > 0
        dg.free()
