"""Shared levels whose total weight (slots, and five for each row) passes 32
bits: a hub's long list scanned by all rows of a large table.  Rows, counts
and digests against the construction and the per-level kernels."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is loaded before the library)

import workloads as w

pytestmark = pytest.mark.gpu

QUERY = w.make_query([0, 1, 2], [(0, 1), (0, 2)], [0, 1])


def two_fans(f0, f1, asked, others):
    """A hub with f0 neighbours x by edges of label 0 and f1 neighbours y by
    edges of label 1, every (f1 // asked)-th y with the label that the query
    asks for; `others` vertices of the hub's label without edges."""
    hub = others // 2
    x = others + 1 + np.arange(f0)
    y = others + 1 + f0 + np.arange(f1)
    want = y[::f1 // asked][:asked]
    vl = np.concatenate([np.zeros(others + 1), np.ones(f0), np.full(f1, 3)]).astype(np.int64)
    vl[want] = 2
    to = np.concatenate([x, y])
    g = w.make_graph(len(vl), vl, np.stack([np.full(len(to), hub), to], 1), [0] * f0 + [1] * f1, "two fans")
    rows = np.stack([np.full(f0 * asked, hub), np.repeat(x, asked), np.tile(want, f0)], 1) if asked < 10 else None
    return g, rows


# the second level weighs f0 (f1 + 5): 2^32 - 1, 2^32, 2^32 + 65,530, 2^32 from a
# list of half a share's limit, and 2^32 + 24,576 of lists clamped at 2^20 + 1
@pytest.mark.parametrize("f0,f1", [(65535, 65532), (65536, 65531), (65534, 65534), (8192, 524283), (4096, 1 << 21)])
def test_total_weight_past_32_bits(f0, f1):
    import paper_1906_03420_amd as gsi
    g, want = two_fans(f0, f1, 3, 1099)  # 1,100 roots: the first level is shared too
    flags = gsi.GSI_FILTER_LABEL_ONLY | gsi.GSI_NO_CHUNKS
    print(f0, f1, flush=True)
    with gsi.Context(gsi.gsi_graph_bytes_needed(g.n, g.m) + (4 << 30)) as ctx:
        dg = ctx.load(g)
        base = dg.query(QUERY, flags=flags | gsi.GSI_NO_FUSED, order=[0, 1, 2])
        np.testing.assert_array_equal(base.rows(), want)
        for extra in (0, gsi.GSI_COUNT_ONLY, gsi.GSI_HOMOMORPHISM):
            r = dg.query(QUERY, flags=flags | extra, order=[0, 1, 2])
            assert r.count == len(want) and r.digest == base.digest
            assert r.stats()["survivors"][1:] == [f0, len(want)]
            if not extra & gsi.GSI_COUNT_ONLY:
                np.testing.assert_array_equal(r.rows(), want)
            r.free()
        base.free()
        dg.free()


@pytest.mark.parametrize("copies", [1, 2])
def test_total_weight_past_32_bits_in_a_batch(copies):
    """Every y asked for: 65,534^2 rows, counted."""
    import paper_1906_03420_amd as gsi
    f = 65534
    g, _ = two_fans(f, f, f, 0)
    print(copies, flush=True)
    with gsi.Context(gsi.gsi_graph_bytes_needed(g.n, g.m) + (8 << 30)) as ctx:
        dg = ctx.load(g)
        base = dg.query(QUERY, flags=gsi.GSI_COUNT_ONLY | gsi.GSI_NO_FUSED)
        assert base.count == f * f
        b = dg.batch([QUERY] * copies, flags=gsi.GSI_COUNT_ONLY)
        counts, digests = b.results()
        assert counts.tolist() == [f * f] * copies
        assert [tuple(int(t) for t in d) for d in digests] == [base.digest] * copies
        b.free()
        base.free()
        dg.free()
