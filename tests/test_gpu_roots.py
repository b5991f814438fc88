"""The candidate counts and the root table on both sides of the bitset length
(2^20 vertices) from which they are counted and emitted in grid-wide runs."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is loaded before the library)

import workloads as w

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [63, 64, 4096 * 64 + 1, 1 << 20, (1 << 20) + 1, (1 << 20) + 64 * 63 + 5, 5_000_077])
def test_roots_and_counts(n):
    import paper_1906_03420_amd as gsi
    r = np.random.default_rng(n)
    vl = r.integers(0, 5, n)
    vl[n - 1] = 0
    a = np.arange(0, n - 1, 2)  # a matching: vertex 2i with 2i + 1
    g = w.make_graph(n, vl, np.stack([a, a + 1], 1), r.integers(0, 2, len(a)), "roots")
    print(n, flush=True)
    with gsi.Context(gsi.gsi_graph_bytes_needed(g.n, g.m) + (1 << 30)) as ctx:
        dg = ctx.load(g)
        for lab in (0, 4):
            res = dg.query(w.make_query([lab], [], []))
            np.testing.assert_array_equal(res.rows()[:, 0], np.nonzero(vl == lab)[0])
            res.free()
        # an edge with label 1 between labels 0 and 3, and the reverse row order
        el = np.zeros(n, np.int64)
        el[a] = g.elabel
        lo = a[(g.elabel == 1) & (vl[a] == 0) & (vl[a + 1] == 3)]
        hi = a[(g.elabel == 1) & (vl[a] == 3) & (vl[a + 1] == 0)]
        want = np.concatenate([np.stack([lo, lo + 1], 1), np.stack([hi + 1, hi], 1)])
        want = want[np.argsort(want[:, 0])]
        for flags in (0, gsi.GSI_NO_FUSED, gsi.GSI_FILTER_LABEL_ONLY, gsi.GSI_HOMOMORPHISM):
            q = w.make_query([0, 3], [(0, 1)], [1])
            res = dg.query(q, flags=flags)
            np.testing.assert_array_equal(res.sorted_rows(), want)
            res.free()
        bits, cnt = dg.filter(w.make_query([0, 3], [(0, 1)], [1]))
        assert cnt.tolist() == [int(np.unpackbits(x.view(np.uint8)).sum()) for x in bits]
        dg.free()
