"""Per-level joins launched before |GBA| is known: levels at, below and past
what the launch was sized for, rows found by 64-way rounds over tables of one
to 10^5 rows with empty lists among them, scans of one to five rounds."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is loaded before the library)

import workloads as w

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb,nc,gap", [(256, 256, 0), (256, 257, 0), (257, 256, 3), (300, 400, 2), (1, 70_000, 0),
                                       (70_000, 1, 0), (70_000, 2, 5), (8193, 3, 4), (33_000, 1, 2), (4097, 1, 7)])
def test_level_sizes(nb, nc, gap):
    """Roots a_i - b_i (label 0), b_i - c_ij (label 1): one slot per row at the
    first level, nc at the second; every gap-th b has no c."""
    import paper_1906_03420_amd as gsi
    a = np.arange(nb)
    b = nb + a
    keep = np.ones(nb, bool) if not gap else (a % gap != 0)
    owner = np.repeat(b[keep], nc)
    c = 2 * nb + np.arange(len(owner))
    e = np.concatenate([np.stack([a, b], 1), np.stack([owner, c], 1)])
    vl = np.concatenate([np.zeros(nb), np.ones(nb), np.full(len(c), 2)]).astype(np.int64)
    g = w.make_graph(2 * nb + len(c), vl, e, [0] * nb + [1] * len(c), "two levels")
    q = w.make_query([0, 1, 2], [(0, 1), (1, 2)], [0, 1])
    order = [0, 1, 2]
    want = np.stack([owner - nb, owner, c], 1)
    print(nb, nc, gap, flush=True)
    with gsi.Context(gsi.gsi_graph_bytes_needed(g.n, g.m) + (1 << 30)) as ctx:
        dg = ctx.load(g)
        for flags in (gsi.GSI_NO_FUSED | gsi.GSI_FILTER_LABEL_ONLY, gsi.GSI_NO_FUSED | gsi.GSI_NO_LIST_FILTER, 0,
                      gsi.GSI_NO_CHUNKS | gsi.GSI_FILTER_LABEL_ONLY):
            for o in (order, None):
                r = dg.query(q, flags=flags, order=o)
                assert r.count == len(want)
                np.testing.assert_array_equal(r.sorted_rows(), want)
                st = r.stats()
                if o is not None and flags & gsi.GSI_NO_FUSED and flags & gsi.GSI_FILTER_LABEL_ONLY:
                    assert st["gba"][1:] == [nb, len(c)] and st["survivors"][1:] == [nb, len(c)]
                r.free()
        dg.free()


def test_multi_more_labelled_edges_than_vertices():
    """Eight labels on every pair of a two-vertex query: more linking edges
    than placed vertices, over a table of thousands of rows."""
    import paper_1906_03420_amd as gsi
    n = 3000
    edges = [(i, (i + 1) % n, l) for i in range(n) for l in range(8)]
    g = w.make_mgraph(n, [[0]] * n, edges, "eight labels")
    q = w.make_mquery([[0], [0]], [(0, 1, l) for l in range(8)])
    i = np.arange(n)
    want = np.concatenate([np.stack([i, (i + 1) % n], 1), np.stack([(i + 1) % n, i], 1)])
    with gsi.Context(1 << 30) as ctx:
        dg = ctx.load_multi(g)
        r = dg.query_multi(q)
        assert r.count == 2 * n
        np.testing.assert_array_equal(r.sorted_rows(), want[np.lexsort((want[:, 1], want[:, 0]))])
        r.free()
        dg.free()
