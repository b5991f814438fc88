"""Batch queries that several workgroups run and do not finish: passes with
more workgroups from the table reached, the engine from there, and, where the
arena is short, from the roots again.  Counts, digests and rows against the
per-level kernels and the construction."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is loaded before the library)

import workloads as w

pytestmark = pytest.mark.gpu


def layers(roots, fans):
    """A vertex of layer i has fans[i] neighbours of its own in layer i + 1, by
    edges of label i; vertices have their layer's label.  Also every path from
    the first layer to the last."""
    first, paths, edges, labels, vl = 0, np.arange(roots)[:, None], [], [], [np.zeros(roots, np.int64)]
    for i, f in enumerate(fans):
        n = len(paths)
        first += n
        new = first + np.arange(n * f)
        edges.append(np.stack([np.repeat(paths[:, -1], f), new], 1))
        labels += [i] * (n * f)
        vl.append(np.full(n * f, i + 1))
        paths = np.concatenate([np.repeat(paths, f, 0), new[:, None]], 1)
    return w.make_graph(first + len(paths), np.concatenate(vl), np.concatenate(edges), labels, "layers"), paths


def path_query(n):
    return w.make_query(list(range(n)), [(i, i + 1) for i in range(n - 1)], list(range(n - 1)))


# the second level has more survivors than any cluster's table (the engine goes
# on at it, then at the third); more slots than 32 or 16 workgroups hold, not 64;
# fits at once; a first level past one workgroup, the second past all
CASES = [(400, [20, 40, 4]), (100, [50, 140, 1, 2]), (120, [40, 10, 3]), (60, [300, 60, 1])]


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("copies", [1, 3, 8, 20])
def test_batches_left_by_clusters(case, copies):
    import paper_1906_03420_amd as gsi
    g, paths = layers(*CASES[case])
    k = paths.shape[1]
    long, short = path_query(k), path_query(k - 1)
    print(case, copies, len(paths), flush=True)
    with gsi.Context(gsi.gsi_graph_bytes_needed(g.n, g.m) + (8 << 30)) as ctx:
        dg = ctx.load(g)
        want = []
        for q in (long, short):
            r = dg.query(q, flags=gsi.GSI_COUNT_ONLY | gsi.GSI_NO_FUSED)
            want.append((r.count, r.digest))
            r.free()
        assert want[0][0] == len(paths)
        qs = ([long, short] * copies)[:copies + 1]
        for flags in (gsi.GSI_COUNT_ONLY, 0):
            b = dg.batch(qs, flags=flags, threads=256, grid_scale=8)
            for i in range(len(qs)):
                assert (b.count(i), b.digest(i)) == want[i & 1]
            if not flags:
                np.testing.assert_array_equal(b.sorted_rows(0), paths)
                np.testing.assert_array_equal(b.sorted_rows(1), np.unique(paths[:, :-1], axis=0))
            b.free()
        dg.free()


def test_batch_left_by_clusters_in_tight_arenas():
    """Kept results leave the batch less and less room: tables from clusters are
    held, given up for the first query's level, or never made; each arena
    answers right or refuses."""
    import paper_1906_03420_amd as gsi
    g, paths = layers(400, [20, 40, 4])
    q = path_query(4)
    size = gsi.gsi_graph_bytes_needed(g.n, g.m)
    with gsi.Context(size, flags=gsi.GSI_CTX_PROFILE) as ctx:
        dg = ctx.load(g)
        r = dg.query(q, flags=gsi.GSI_COUNT_ONLY | gsi.GSI_NO_FUSED)
        want = (r.count, r.digest)
        r.free()
        kept, seen = [], []
        for free in (800, 500, 300, 200, 150, 120, 100, 90, 80, 70, 60, 50, 45, 40, 35, 30, 25, 20, 15):
            for lab, rows in ((3, len(paths)), (2, len(paths) // 4), (1, 8000)):
                one = w.make_query([lab], [], [])
                while size - ctx.memory()[0] - 4 * rows >= free << 20:
                    kept.append(dg.query(one))
            ctx.kernel_stats_reset()
            try:
                b = dg.batch([q] * 6, flags=gsi.GSI_COUNT_ONLY, threads=256, grid_scale=8)
            except gsi.GsiError as e:
                assert e.status == gsi.GSI_E_NOMEM
                seen.append((free, "refused"))
                continue
            assert all((b.count(i), b.digest(i)) == want for i in range(6))
            b.free()
            ran = {x["name"]: x["launches"] for x in ctx.kernel_stats()}
            seen.append((free, ran.get("k_fused_cluster", 0), ran.get("k_wjoin", 0)))
        print(seen, flush=True)
        assert seen[0][1:] == (1, 2)  # one pass, then the engine's last two levels
        for r in kept:
            r.free()
        dg.free()
