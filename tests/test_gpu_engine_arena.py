"""The level-synchronous engine in arenas around the least that holds a step
with filtered lists: allocations that fail before, between and after the
step's uploads leave it in order; every arena gives the right answer or is
refused, and none is refused above one that was enough."""
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
