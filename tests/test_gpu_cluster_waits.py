"""Workgroups that share levels when some of them are missing: helpers that
never check in, waits that run out, and a helper that leaves at each of a
query's meetings.  Every kernel ends by itself; rows, order and digests are the
per-level kernels'."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is loaded before the library)

import workloads as w

pytestmark = pytest.mark.gpu


def quit_at(n):
    return n << 16


def tree(roots, fans):
    """Layer i's vertices have fans[i] neighbours each (a number, or one per
    vertex) of their own in layer i + 1; labels as the layers."""
    first, last, edges, labels, vl = 0, np.arange(roots), [], [], [np.zeros(roots, np.int64)]
    for i, f in enumerate(fans):
        f = np.broadcast_to(f, len(last))
        first += len(last)
        new = first + np.arange(int(f.sum()))
        edges.append(np.stack([np.repeat(last, f), new], 1))
        labels += [i] * len(new)
        vl.append(np.full(len(new), i + 1))
        last = new
    n, k = first + len(last), len(fans) + 1
    g = w.make_graph(n, np.concatenate(vl), np.concatenate(edges), labels, "tree")
    return g, w.make_query(list(range(k)), [(i, i + 1) for i in range(k - 1)], list(range(k - 1)))


def hubs(n, small, big, every):
    f = np.full(n, small)
    f[::every] = big
    return f


# parts left as they are; slots dealt out anew (hubs)
TREES = [(1500, (3, 5, 2)), (1500, (hubs(1500, 2, 7000, 1500), hubs(9998, 1, 4000, 3000), 2))]


def joins(ctx):
    return sum(s["launches"] for s in ctx.kernel_stats() if s["name"] == "k_join")


@pytest.mark.parametrize("which", range(len(TREES)))
def test_a_helper_leaves(which):
    import paper_1906_03420_amd as gsi
    g, q = tree(*TREES[which])
    order = list(range(q.k))
    left = []
    for mode in [0] + [quit_at(n) for n in range(1, 16)] + [gsi.GSI_CTX_TEST_SHORT_WAITS, gsi.GSI_CTX_TEST_NO_HELPERS]:
        print(which, hex(mode), flush=True)
        with gsi.Context(gsi.gsi_graph_bytes_needed(g.n, g.m) + (4 << 30), flags=gsi.GSI_CTX_PROFILE | mode) as ctx:
            dg = ctx.load(g)
            if mode == 0:
                r = dg.query(q, flags=gsi.GSI_NO_FUSED, order=order)
                rows, digest, stats = r.rows(), r.digest, r.stats()
                r.free()
            ctx.kernel_stats_reset()
            r = dg.query(q, order=order)
            left.append(joins(ctx) > 0)
            assert r.digest == digest
            np.testing.assert_array_equal(r.rows(), rows)
            st = r.stats()
            assert st["rows"][1:] == stats["rows"][1:] and st["survivors"][1:] == stats["survivors"][1:]
            r.free()
            r = dg.query(q, flags=gsi.GSI_COUNT_ONLY, order=order)
            assert (r.count, r.digest) == (len(rows), digest)
            r.free()
            dg.free()
    # three levels of three or four meetings; a level that a helper leaves is
    # given up at that meeting or the next
    assert not left[0] and all(left[1:9]) and not any(left[13:16]) and left[17]


@pytest.mark.parametrize("roots,fan", [(1200, 10), (600, 20), (4096, 4)])
def test_levels_alone_without_helpers(roots, fan):
    """More rows or slots than are run alone when there are helpers, no more than
    one workgroup holds: it runs them when none has checked in."""
    import paper_1906_03420_amd as gsi
    g, q = tree(roots, (fan,))
    with gsi.Context(gsi.gsi_graph_bytes_needed(g.n, g.m) + (4 << 30),
                     flags=gsi.GSI_CTX_PROFILE | gsi.GSI_CTX_TEST_NO_HELPERS) as ctx:
        dg = ctx.load(g)
        base = dg.query(q, flags=gsi.GSI_NO_FUSED, order=[0, 1])
        ctx.kernel_stats_reset()
        r = dg.query(q, order=[0, 1])
        assert joins(ctx) == 0 and r.digest == base.digest
        np.testing.assert_array_equal(r.rows(), base.rows())
        r.free()
        base.free()
        dg.free()


@pytest.mark.parametrize("copies", [1, 5, 20])
def test_a_helper_leaves_in_a_batch(copies):
    import paper_1906_03420_amd as gsi
    g, q = tree(*TREES[1])
    for mode in [0] + [quit_at(n) for n in range(1, 16)] + [gsi.GSI_CTX_TEST_SHORT_WAITS, gsi.GSI_CTX_TEST_NO_HELPERS]:
        print(copies, hex(mode), flush=True)
        with gsi.Context(gsi.gsi_graph_bytes_needed(g.n, g.m) + (4 << 30), flags=mode) as ctx:
            dg = ctx.load(g)
            if mode == 0:
                r = dg.query(q, flags=gsi.GSI_NO_FUSED)
                rows, digest = r.sorted_rows(), r.digest
                r.free()
            for flags in (gsi.GSI_COUNT_ONLY, 0):
                b = dg.batch([q] * copies, flags=flags, threads=256, grid_scale=8)
                for i in range(copies):
                    assert (b.count(i), b.digest(i)) == (len(rows), digest)
                if not flags:
                    np.testing.assert_array_equal(b.sorted_rows(copies - 1), rows)
                b.free()
            dg.free()
