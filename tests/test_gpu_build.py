"""Graph build at the sizes where its kernels change path: the edges of the
sort's, the signatures' and the runs' tiles, hubs and isolated ids across
tiles, the two widths of the sort's tiles, and entries that do not pack into
64 bits.  Integer work, compared bit for bit with numpy."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is loaded before the library)

from oracle import spec
import workloads as w

pytestmark = pytest.mark.gpu


def _graph(name, n, m, nvl, nel, seed):
    """A simple graph of m edges in no particular order."""
    r = np.random.default_rng(seed)
    if name == "star":  # one vertex with every entry of many tiles
        a = np.zeros(m, np.int64)
        b = np.arange(1, m + 1)
    elif name == "matching":  # every vertex has one entry
        a = np.arange(m) * 2
        b = a + 1
    else:  # random pairs, ids spread over [0, n)
        a = r.integers(0, n, 2 * m + 16)
        b = r.integers(0, n, 2 * m + 16)
        keys = np.unique(np.minimum(a, b)[a != b].astype(np.int64) << 32 | np.maximum(a, b)[a != b])
        keys = r.permutation(keys)[:m]
        a, b = keys >> 32, keys & 0xFFFFFFFF
    p = r.permutation(len(a))
    flip = r.random(len(a)) < 0.5
    a, b = np.where(flip, b, a)[p], np.where(flip, a, b)[p]
    return w.make_graph(n, r.integers(0, nvl, n), np.stack([a, b], 1), r.integers(0, nel, len(a)), name)


def _check(dg, g, sig=True):
    s = np.concatenate([g.src, g.dst]).astype(np.int64)
    d = np.concatenate([g.dst, g.src]).astype(np.int64)
    l = np.concatenate([g.elabel, g.elabel]).astype(np.int64)
    info = dg.info()
    assert info["n_edge_labels"] == (int(g.elabel.max()) + 1 if g.m else 0)
    groups = 0
    order = np.lexsort((d, s, l))
    s, d, l = s[order], d[order], l[order]
    for lab in np.unique(l).tolist():
        lo, hi = np.searchsorted(l, [lab, lab + 1])
        gl, ci = dg.pcsr(lab)
        keys, offs = gl[:, 0:30:2], gl[:, 1:32:2].astype(np.int64)
        # lists lie in group, then slot order, without gaps
        flat = offs.ravel()
        assert flat[0] == 0 and np.all(np.diff(flat) >= 0) and flat[-1] == len(ci) == hi - lo
        lens = np.diff(offs, axis=1)
        used = keys != 0xFFFFFFFF
        assert np.all(lens[~used] == 0)
        owner = np.repeat(keys[used].astype(np.int64), lens[used])
        at = np.argsort(owner, kind="stable")
        np.testing.assert_array_equal(owner[at], s[lo:hi])
        np.testing.assert_array_equal(ci[at], d[lo:hi])
        assert len(gl) == len(np.unique(s[lo:hi])) == used.sum()
        groups += len(gl)
    assert info["total_groups"] == groups
    if not sig:
        return
    got = dg.signatures()
    np.testing.assert_array_equal(got[0], g.vlabel)
    key, cnt = np.unique(s * 240 + spec.signature_group(l, g.vlabel[d]).astype(np.int64), return_counts=True)
    v, grp = key // 240, key % 240
    want = np.zeros(15 * g.n, np.uint32)
    np.bitwise_or.at(want, (grp // 16) * g.n + v, np.where(cnt > 1, 3, 1).astype(np.uint32) << (2 * (grp % 16)).astype(np.uint32))
    np.testing.assert_array_equal(got[1:].ravel(), want)


@pytest.mark.parametrize("name,n,m,nvl,nel", [
    ("random", 2, 1, 1, 1), ("random", 300, 1023, 3, 1), ("random", 300, 1024, 3, 2), ("random", 300, 1025, 3, 2),
    ("random", 1000, 2047, 5, 3), ("random", 1000, 2049, 5, 300), ("random", 500, 4097, 2, 4),
    ("random", 1 << 20, 3000, 40, 5), ("star", 20_000, 19_999, 7, 3), ("star", 5000, 2048, 2, 1),
    ("matching", 40_000, 20_000, 9, 2), ("random", 70_000, 200_001, 300, 20)])
def test_build_at_tile_edges(name, n, m, nvl, nel):
    import paper_1906_03420_amd as gsi
    g = _graph(name, n, m, nvl, nel, 5)
    print(name, n, m, nvl, nel, flush=True)
    with gsi.Context(gsi.gsi_graph_bytes_needed(g.n, g.m) + (64 << 20)) as ctx:
        dg = ctx.load(g)
        _check(dg, g)
        dg.free()


@pytest.mark.parametrize("m", [(1 << 22) - 1, 1 << 22])
def test_build_on_both_sides_of_the_wide_sort(m):
    import paper_1906_03420_amd as gsi
    g = _graph("random", 1_500_000, m, 32, 3, 6)
    print(g.n, g.m, flush=True)
    with gsi.Context(gsi.gsi_graph_bytes_needed(g.n, g.m) + (64 << 20)) as ctx:
        dg = ctx.load(g)
        _check(dg, g)
        dg.free()


def test_build_of_entries_past_64_bits():
    """26 bits an end and 16 bits of label: sorted as three arrays."""
    import paper_1906_03420_amd as gsi
    g = _graph("random", (1 << 25) + 5, 9000, 3, 2, 7)
    g.elabel[:] = g.elabel * 65535
    with gsi.Context(gsi.gsi_graph_bytes_needed(g.n, g.m) + (64 << 20)) as ctx:
        dg = ctx.load(g)
        _check(dg, g)
        dg.free()


@pytest.mark.parametrize("n,m", [(1000, 5000), ((1 << 25) + 5, 5000)])
def test_repeated_pair_is_refused(n, m):
    """Also when the repeated pair's labels differ and its ends are swapped."""
    import paper_1906_03420_amd as gsi
    g = _graph("random", n, m, 3, 2, 8)
    g.elabel[0], g.elabel[m - 1] = 0, 65535 if n > 1000 else 1
    g.src[m - 1], g.dst[m - 1] = g.dst[0], g.src[0]
    with gsi.Context(gsi.gsi_graph_bytes_needed(g.n, g.m) + (64 << 20)) as ctx:
        with pytest.raises(gsi.GsiError, match="repeated vertex pair"):
            ctx.load(g)
