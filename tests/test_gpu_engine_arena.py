"""The level-synchronous engine in arenas around the least that holds a step
with filtered lists: allocations that fail before, between and after the
step's uploads leave it in order; every arena gives the right answer or is
refused, and none is refused above one that was enough."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is loaded before the library)

import workloads as w

pytestmark = pytest.mark.gpu


def test_filtered_steps_in_tight_arenas():
    import paper_1906_03420_amd as gsi
    n, k = 44, 5
    g = w.complete_graph(n)
    q = w.make_query([0] * k, [(i, i + 1) for i in range(k - 1)], [0] * (k - 1))
    want = 1
    for i in range(k):
        want *= n - i
    flags = gsi.GSI_COUNT_ONLY | gsi.GSI_BATCH_LEVELS_ONLY

    def run(kib, copies=1, profile=False):
        with gsi.Context(kib << 10, flags=gsi.GSI_CTX_PROFILE if profile else 0) as ctx:
            dg = ctx.load(g)
            ctx.kernel_stats_reset()
            try:
                b = dg.batch([q] * copies, flags=flags, threads=256, grid_scale=8)
            except gsi.GsiError as e:
                assert e.status == gsi.GSI_E_NOMEM
                return False
            counts, digests = b.results()
            assert counts.tolist() == [want] * copies
            assert len({tuple(int(t) for t in d) for d in digests}) == 1
            b.free()
            if profile:
                assert {x["name"]: x["launches"] for x in ctx.kernel_stats()}.get("k_fn_bits", 0) > 0
            return True

    lo, hi = 16 << 10, 4 << 20
    assert run(hi, 2, True) and not run(lo)
    while hi - lo > 64:
        mid = (lo + hi) // 2
        if run(mid):
            hi = mid
        else:
            lo = mid
    print("least arena", hi, "KiB", flush=True)
    for step in (64, 97, 1021, 4099):
        for t in range(1, 9):
            assert run(hi + t * step)
            run(hi - t * step)
    # several queries, whose tables wait while others advance: a step of all, of
    # half of them, of one, or refused; there is room for all in the end
    assert any([run(hi + t * hi // 4, 3) for t in range(1, 17)])


def test_step_that_fits_without_filtered_lists_only():
    """28 a's joined to 160,000 b's, each b to eight c's of which one is asked
    for, and that one to a w.  At the c's a table of 4.48 * 10^6 rows scans
    eight elements each, fourteen times the label's entries, so the lists are
    filtered (11 MB); the next table takes 54 MB.  Kept results fill the arena
    up to 243.5 MB, in which the step fits without them."""
    import paper_1906_03420_amd as gsi
    na, nb, dc, free = 28, 160_000, 8, 243_500_000
    b = na + np.arange(nb)
    c = na + nb + np.arange(nb * dc)
    x = na + nb + nb * dc + np.arange(nb)
    e = np.concatenate([np.stack([np.repeat(np.arange(na), nb), np.tile(b, na)], 1),
                        np.stack([np.repeat(b, dc), c], 1), np.stack([c[::dc], x], 1)])
    vl = np.concatenate([np.zeros(na), np.ones(nb), np.where(np.arange(nb * dc) % dc == 0, 2, 4), np.full(nb, 3)])
    g = w.make_graph(len(vl), vl.astype(np.int64), e, [0] * (na * nb) + [1] * (nb * dc) + [2] * nb, "three levels")
    q = w.make_query([0, 1, 2, 3], [(0, 1), (1, 2), (2, 3)], [0, 1, 2])
    size = gsi.gsi_graph_bytes_needed(g.n, g.m)
    with gsi.Context(size) as ctx:
        dg = ctx.load(g)
        want = dg.query(q, flags=gsi.GSI_COUNT_ONLY)
        digest = want.digest
        assert want.count == na * nb
        want.free()
        kept = []
        for lab, rows in ((4, nb * (dc - 1)), (1, nb), (0, na)):
            one = w.make_query([lab], [], [])
            while size - ctx.memory()[0] - 4 * rows >= free:
                kept.append(dg.query(one))
                assert kept[-1].count == rows
        out = dg.batch([q], flags=gsi.GSI_COUNT_ONLY | gsi.GSI_BATCH_LEVELS_ONLY, threads=256, grid_scale=8)
        assert out.count(0) == na * nb and out.digest(0) == digest
        out.free()
        for r in kept:
            r.free()
        dg.free()
