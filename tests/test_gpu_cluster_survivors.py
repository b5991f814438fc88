"""Levels of few enough slots for one workgroup, but with more survivors than
its tables hold: the helpers are called to them."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is loaded before the library)

import workloads as w

pytestmark = pytest.mark.gpu


# 4,096, 4,200 and 8,000 survivors of a first level, 4,800 of a second one (roots
# enough for the first launch to have helpers)
@pytest.mark.parametrize("roots,fans", [(512, (8, 3)), (280, (15, 3)), (400, (20, 3)), (600, (1, 8, 2))])
def test_more_survivors_than_one_workgroup_holds(roots, fans):
    import paper_1906_03420_amd as gsi
    paths, first, edges, labels, vl = np.arange(roots)[:, None], 0, [], [], [np.zeros(roots, np.int64)]
    for i, f in enumerate(fans):
        first += len(paths)
        new = first + np.arange(len(paths) * f)
        edges.append(np.stack([np.repeat(paths[:, -1], f), new], 1))
        labels += [i] * len(new)
        vl.append(np.full(len(new), i + 1))
        paths = np.concatenate([np.repeat(paths, f, 0), new[:, None]], 1)
    g = w.make_graph(first + len(paths), np.concatenate(vl), np.concatenate(edges), labels, "layers")
    k = len(fans) + 1
    q = w.make_query(list(range(k)), [(i, i + 1) for i in range(k - 1)], list(range(k - 1)))
    print(roots, fans, flush=True)
    with gsi.Context(gsi.gsi_graph_bytes_needed(g.n, g.m) + (4 << 30), flags=gsi.GSI_CTX_PROFILE) as ctx:
        dg = ctx.load(g)
        for extra in (0, gsi.GSI_COUNT_ONLY, gsi.GSI_HOMOMORPHISM):
            ctx.kernel_stats_reset()
            r = dg.query(q, flags=extra, order=list(range(k)))
            assert r.count == len(paths)
            if not extra & gsi.GSI_COUNT_ONLY:
                np.testing.assert_array_equal(r.rows(), paths)
            r.free()
            assert not any(x["name"].startswith("k_join") for x in ctx.kernel_stats() if x["launches"])
        dg.free()
