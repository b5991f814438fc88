"""Levels that the single-query workgroup shares with its helpers: sizes at and
past what it runs alone, what a workgroup's share holds, what the tables and
the result hold; shares without rows; queries expected to be too small for
helpers.  Rows are compared in order with the per-level kernels' and with
their construction."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is loaded before the library)

import workloads as w

pytestmark = pytest.mark.gpu


def chain(fans, every, singles=0):
    """a_i - b_i (label 0), b_i - its fans[i] c's (label 1), every `every`-th c
    - d (label 2); `singles` pairs of other vertices with label 1."""
    nb = len(fans)
    a = np.arange(nb)
    b = nb + a
    owner = np.repeat(b, fans)
    nc = len(owner)
    c = 2 * nb + np.arange(nc)
    tail = c[::every]
    d = 2 * nb + nc + np.arange(len(tail))
    s = 2 * nb + nc + len(tail) + np.arange(2 * singles)
    e = np.concatenate([np.stack([a, b], 1), np.stack([owner, c], 1), np.stack([tail, d], 1), s.reshape(-1, 2)])
    lab = [0] * nb + [1] * nc + [2] * len(tail) + [1] * singles
    vl = np.repeat([0, 1, 2, 3, 4], [nb, nb, nc, len(tail), 2 * singles])
    g = w.make_graph(len(vl), vl, e, lab, "chain")
    want = np.stack([owner[::every] - nb, owner[::every], tail, d], 1)
    return g, want, nc


CASES = [
    ([64] * 64, 1, 0), ([241] * 17, 1, 0),             # 4096 and 4097 slots
    ([4] * 1024, 1, 0), ([4] * 1025, 1, 0),            # 1024 and 1025 rows
    ([2] * 4096, 1, 0), ([1] * 4097, 1, 0),            # rows one workgroup can hold, one more
    ([1] * 32768, 3, 0), ([1] * 32769, 3, 0),          # roots the kernel is given, one more
    ([1000] * 5, 1, 0), ([6000] + [0] * 99, 2, 0),     # shares without rows, without slots
    ([16384], 1, 0), ([16385], 1, 0), ([20000, 3], 1, 0),  # slots one share can hold
    ([16] * 8192, 64, 0), ([130] * 1025, 40, 0),       # 131072 rows of a table and more
    ([120] * 1090, 1, 0), ([16] * 8192, 1, 0),
    ([6000], 1, 30000), ([10000] * 2, 1, 60000), ([40] * 300, 1, 100000),  # expected small
    ([128] * 64, 1, 0), ([241] * 34, 1, 0),            # 8192 and 8194 slots
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_shared_levels(case):
    import paper_1906_03420_amd as gsi
    fans, every, singles = CASES[case]
    g, want, nc = chain(np.asarray(fans), every, singles)
    path4 = w.make_query([0, 1, 2, 3], [(0, 1), (1, 2), (2, 3)], [0, 1, 2])
    path3 = w.make_query([0, 1, 2], [(0, 1), (1, 2)], [0, 1])
    flags = gsi.GSI_FILTER_LABEL_ONLY | gsi.GSI_NO_CHUNKS
    print(case, len(fans), nc, len(want), flush=True)
    with gsi.Context(gsi.gsi_graph_bytes_needed(g.n, g.m) + (4 << 30)) as ctx:
        dg = ctx.load(g)
        for q, k in ((path4, 4), (path3, 3)):
            base = dg.query(q, flags=flags | gsi.GSI_NO_FUSED, order=list(range(k)))
            ref, digest, levels = base.rows(), base.digest, base.stats()
            if k == 4:
                np.testing.assert_array_equal(ref, want)
            else:
                assert base.count == nc
            base.free()
            for extra in (0, gsi.GSI_COUNT_ONLY, gsi.GSI_HOMOMORPHISM):
                r = dg.query(q, flags=flags | extra, order=list(range(k)))
                st = r.stats()
                assert r.count == len(ref) and r.digest == digest
                assert st["rows"][1:] == levels["rows"][1:]
                assert st["survivors"][1:] == levels["survivors"][1:]
                if not extra & gsi.GSI_COUNT_ONLY:
                    np.testing.assert_array_equal(r.rows(), ref)
                r.free()
        dg.free()


def test_shared_last_level_past_the_result_rows():
    """A last level of more rows than the kernel's result holds, and one of
    exactly as many."""
    import paper_1906_03420_amd as gsi
    q = w.make_query([0, 1, 2], [(0, 1), (1, 2)], [0, 1])
    for nb, fan in ((1024, 256), (1041, 252)):
        g, _, nc = chain(np.full(nb, fan), 1)
        assert (nc > 262144) == (nb == 1041)
        print(nb, fan, flush=True)
        with gsi.Context(gsi.gsi_graph_bytes_needed(g.n, g.m) + (4 << 30)) as ctx:
            dg = ctx.load(g)
            flags = gsi.GSI_FILTER_LABEL_ONLY | gsi.GSI_NO_CHUNKS
            a = dg.query(q, flags=flags | gsi.GSI_NO_FUSED, order=[0, 1, 2])
            b = dg.query(q, flags=flags, order=[0, 1, 2])
            assert a.count == b.count == nc and a.digest == b.digest
            np.testing.assert_array_equal(a.rows(), b.rows())
            a.free()
            b.free()
            dg.free()


# (copies of the queries, chain): the most copies with several workgroups each
# and one more, levels that fit only with more CUs per query, and none that fit
@pytest.mark.parametrize("copies,case", [(1, 3), (1, 11), (2, 14), (5, 12), (16, 4), (16, 14), (9, 6), (16, 1), (17, 1),
                                         (17, 5), (2, 17), (1, 15)])
def test_batch_queries_with_several_workgroups(copies, case):
    import paper_1906_03420_amd as gsi
    fans, every, singles = CASES[case]
    g, want, _ = chain(np.asarray(fans), every, singles)
    two = [w.make_query([0, 1, 2, 3], [(0, 1), (1, 2), (2, 3)], [0, 1, 2]),
           w.make_query([3, 2, 1], [(0, 1), (1, 2)], [2, 1])]
    qs = two * copies
    exact = [want[np.lexsort(want.T[::-1])]]
    short = want[:, [3, 2, 1]]
    exact.append(short[np.lexsort(short.T[::-1])])
    print(copies, case, len(want), flush=True)
    with gsi.Context(gsi.gsi_graph_bytes_needed(g.n, g.m) + (8 << 30)) as ctx:
        dg = ctx.load(g)
        for threads in (64, 256, 1024):
            for flags in (0, gsi.GSI_COUNT_ONLY):
                b = dg.batch(qs, flags=flags, threads=threads, grid_scale=8)
                info = b.info()
                assert info["empty"] + info["tier1"] + info["tier2"] + info["per_level"] == len(qs)
                for i in range(len(qs)):
                    assert b.count(i) == len(want) and b.digest(i) == b.digest(i & 1)
                    if not flags and i < 4:
                        np.testing.assert_array_equal(b.sorted_rows(i), exact[i & 1])
                if flags == 0:
                    digests = [b.digest(0), b.digest(1)]
                assert [b.digest(0), b.digest(1)] == digests
                b.free()
        dg.free()
