"""The level that a fused workgroup stops at is handed on with its true size:
the join that takes it is launched once."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is loaded before the library)

import workloads as w

pytestmark = pytest.mark.gpu


# lists at the most slots one workgroup joins, past it, past the 65,536 slots
# that the join is launched for at least, and past 2^20
@pytest.mark.parametrize("fan", [16384, 16385, 65536, 65537, 100_000, 1_100_000])
@pytest.mark.parametrize("edges", [1, 2])
def test_level_of_one_long_list(fan, edges):
    """A hub a - b_i, and with two edges a - x - b_i as well; b_i - c_i."""
    import paper_1906_03420_amd as gsi
    b, c, x = 1 + np.arange(fan), 1 + fan + np.arange(fan), 1 + 2 * fan
    e = [np.stack([np.zeros(fan, np.int64), b], 1), np.stack([b, c], 1)]
    lab = [0] * fan + [1] * fan
    pairs, ql = [(0, 1), (1, 2)], [0, 1]
    if edges == 2:
        e += [np.array([[0, x]]), np.stack([np.full(fan, x), b], 1)]
        lab += [2] + [3] * fan
    g = w.make_graph(x + 1, np.repeat([0, 1, 2, 3], [1, fan, fan, 1]), np.concatenate(e), lab, "long list")
    q = w.make_query([0, 1, 2], pairs, ql) if edges == 1 else \
        w.make_query([0, 1, 2, 3], pairs + [(0, 3), (3, 1)], ql + [2, 3])
    order = [0, 1, 2] if edges == 1 else [0, 3, 1, 2]
    want = np.stack([np.zeros(fan, np.int64), b, c] + ([np.full(fan, x)] if edges == 2 else []), 1)
    print(fan, edges, flush=True)
    with gsi.Context(gsi.gsi_graph_bytes_needed(g.n, g.m) + (4 << 30), flags=gsi.GSI_CTX_PROFILE) as ctx:
        dg = ctx.load(g)
        ctx.kernel_stats_reset()
        r = dg.query(q, order=order)
        np.testing.assert_array_equal(r.rows(), want)
        levels = r.stats()["gba"]
        assert levels[order.index(1)] == fan
        r.free()
        joins = sum(s["launches"] for s in ctx.kernel_stats() if s["name"] == "k_join")
        # the long level (16,384 survivors are too many for one workgroup as well)
        # and, at its slots per row, the last one
        assert joins == 2
        dg.free()
