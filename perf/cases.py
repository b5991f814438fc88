"""Performance cases: the work a user of the library has it do, through the
package's public entry points.

Three things happen to a resident data graph: it is loaded (PCSR and
signatures are built on the device), it answers queries one at a time, and it
answers many at once (a batch, or requests to the serving loop).  The listed
cases take each of them at the sizes of this repository's own workloads (the
1,000-vertex Erdos-Renyi graph, the Barabasi-Albert graph of 10^6 vertices,
the R-MAT graphs of scale 22 and 23, power-law labels, random-walk queries of
4 to 24 vertices), at odd sizes, and with the options a program sets (counts
only, rows in a reproducible order, homomorphism, label sets).  `draw` gives
others of the same ranges.

Graphs and queries are generated here on the GPU.  A data graph is resident:
it depends on the case alone and is kept while cases use it; the queries
depend on the seed.  The cases that load a graph make it from the seed.
A query whose tables would pass the case's row limit is drawn again, by a
counting run with that limit (`max_rows`), as a program with a memory budget
would refuse it.
"""
import collections
import math

import numpy as np
import torch

import paper_1906_03420_amd as gsi

DEV = "cuda"


# ------------------------------------------------------------------ cases
def listed():
    return [
        # One four-vertex query on a graph of 1,000 vertices: the smallest
        # call, launches and waits.
        dict(name="tiny_rows", kind="single", model="er", n=1000, m=5000, nvl=4, nel=2, zipf=False, nq=1, kmin=4,
             kmax=4, shape="walk", count_only=False, chunks=True, homo=False, cap=100_000),
        # An odd-sized graph that fits the caches; rows are kept on the device
        # in a reproducible order (no root chunks).
        dict(name="mid_rows", kind="single", model="ba", n=77_777, m=466_641, nvl=16, nel=4, zipf=True, nq=8, kmin=4,
             kmax=9, shape="mixed", count_only=False, chunks=False, homo=False, cap=1_000_000),
        # A million-vertex graph, walk queries of 6 to 12 vertices one at a
        # time: interactive counting.
        dict(name="ba1m_walk", kind="single", model="ba", n=1_000_000, m=9_999_945, nvl=32, nel=8, zipf=True, nq=16,
             kmin=6, kmax=12, shape="walk", count_only=True, chunks=True, homo=False, cap=20_000_000),
        # The same graph under homomorphism semantics (pattern queries in
        # which two query vertices may meet), short and cyclic.
        dict(name="ba1m_homo", kind="single", model="ba", n=1_000_000, m=9_999_945, nvl=32, nel=8, zipf=True, nq=8,
             kmin=4, kmax=7, shape="walk_cycle", count_only=True, chunks=True, homo=True, cap=20_000_000),
        # The largest graph, twelve-vertex queries with every row written to
        # device memory.
        dict(name="rmat23_rows", kind="single", model="rmat", n=1 << 23, m=100_000_000, nvl=100, nel=20, zipf=True,
             nq=8, kmin=12, kmax=12, shape="walk_dense", count_only=False, chunks=False, homo=False,
             cap=20_000_000),
        # The largest graph, counts only, default route.
        dict(name="rmat23_count", kind="single", model="rmat", n=1 << 23, m=100_000_000, nvl=100, nel=20, zipf=True,
             nq=8, kmin=8, kmax=12, shape="walk_dense", count_only=True, chunks=True, homo=False, cap=60_000_000),
        # Vertices and pairs with several labels (knowledge-graph style).
        dict(name="multi_label", kind="multi", n=50_021, m=300_007, nvl=12, nel=4, nq=6, kmin=4, kmax=7,
             cap=1_000_000),
        # A small batch whose rows the program reads back.
        dict(name="batch48_rows", kind="batch", model="ba", n=77_777, m=466_641, nvl=16, nel=4, zipf=True, nq=48,
             kmin=4, kmax=10, shape="mixed", count_only=False, cap=20_000),
        # A large batch of mixed queries, counts only.
        dict(name="batch1024", kind="batch", model="ba", n=1_000_000, m=9_999_945, nvl=32, nel=8, zipf=True, nq=1024,
             kmin=4, kmax=16, shape="mixed", count_only=True, cap=4_000_000),
        # Requests to the serving loop, all waiting at once.
        dict(name="serve256", kind="serve", model="rmat", n=1 << 22, m=50_000_000, nvl=64, nel=16, zipf=True, nq=256,
             kmin=4, kmax=24, shape="mixed", cap=400_000),
        # A small graph loaded and asked one query: start-up of a program.
        dict(name="load_small", kind="load", model="ba", n=100_003, m=1_000_000, nvl=32, nel=8, zipf=True, kmin=5,
             kmax=5, shape="walk", cap=4_000_000),
        # The largest graph loaded from device arrays and asked one query.
        dict(name="load_rmat23", kind="load", model="rmat", n=1 << 23, m=100_000_000, nvl=100, nel=20, zipf=True,
             kmin=6, kmax=6, shape="walk", cap=20_000_000),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["single", "single", "single", "batch", "batch", "serve", "load", "load", "multi"])
    if kind == "multi":
        n = _log(rng, 2_000, 200_000)
        kmin = rng.randint(3, 6)
        return dict(kind="multi", n=n, m=int(n * rng.uniform(3, 8)), nvl=rng.randint(8, 20), nel=rng.randint(2, 6),
                    nq=rng.randint(1, 8), kmin=kmin, kmax=kmin + rng.randint(0, 2), cap=1_000_000)
    model = rng.choice(["er", "ba", "rmat"])
    n = _log(rng, 1_000, 4_000_000)
    c = dict(kind=kind, model=model, n=n, m=int(n * rng.uniform(4, 12)), nvl=rng.randint(8, 100),
             nel=rng.randint(2, 20), zipf=rng.random() < 0.75)
    kmin = rng.randint(4, 10)
    c.update(kmin=kmin, kmax=kmin + rng.randint(0, 4), shape=rng.choice(["walk", "walk_cycle", "walk_dense", "mixed"]))
    if kind == "single":
        count_only = rng.random() < 0.5
        c.update(nq=rng.randint(1, 12), count_only=count_only, chunks=count_only, homo=rng.random() < 0.25,
                 cap=10_000_000 if count_only else 2_000_000)
    elif kind == "batch":
        c.update(nq=_log(rng, 4, 512), count_only=True, cap=1_000_000)
    elif kind == "serve":
        c.update(nq=_log(rng, 4, 200), cap=200_000)
    else:
        c.update(kmin=4, kmax=6, shape="walk", cap=10_000_000)
    return c


# ----------------------------------------------------------- data graphs
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed & 0x7FFFFFFF)


def _labels(count, nl, zipf, gen):
    """int32 labels 0..nl-1, uniform or with P(i) proportional to (i+1)^-1.1."""
    if not zipf:
        return torch.randint(0, nl, (count,), device=DEV, dtype=torch.int32, generator=gen)
    cdf = torch.cumsum(torch.arange(1, nl + 1, dtype=torch.float64).pow(-1.1), 0)
    cdf = (cdf / cdf[-1]).to(torch.float32).to(DEV)
    x = torch.rand(count, device=DEV, generator=gen)
    return torch.searchsorted(cdf, x).clamp_(max=nl - 1).to(torch.int32)


def _raw_pairs(c, count, gen):
    """About `count` vertex pairs of the case's model; repeats and loops may be among them."""
    n = c["n"]
    if c["model"] == "er":
        return (torch.randint(0, n, (count,), device=DEV, generator=gen),
                torch.randint(0, n, (count,), device=DEV, generator=gen))
    if c["model"] == "ba":
        # every edge's second end is an end of an earlier edge, drawn uniformly
        # (preferential attachment); the draws that land on second ends are
        # followed until they reach a first end
        d = max(1, count // n)
        e = torch.arange(n * d, device=DEV)
        src = e // d
        pick = (torch.rand(n * d, device=DEV, generator=gen, dtype=torch.float64) * (2 * e + 1)).long()
        at = pick.clone()
        for _ in range(64):
            odd = (at & 1) == 1
            at = torch.where(odd, pick[at >> 1], at)
        return src, src[at >> 1]
    r = torch.zeros(count, device=DEV, dtype=torch.int64)
    q = torch.zeros(count, device=DEV, dtype=torch.int64)
    for _ in range(max(1, (n - 1).bit_length())):
        x = torch.rand(count, device=DEV, generator=gen)
        r = (r << 1) | (x >= 0.76).long()
        q = (q << 1) | (((x >= 0.57) & (x < 0.76)) | (x >= 0.95)).long()
    return r % n, q % n


def _edges(c, gen):
    """The case's graph as int32 device arrays: vertex labels, edge ends and edge labels; a simple graph
    whose edges come in no particular order."""
    n, m = c["n"], c["m"]
    keys = torch.empty(0, device=DEV, dtype=torch.int64)
    extra = 1.12 if c["model"] == "rmat" else 1.03
    for _ in range(6):
        a, b = _raw_pairs(c, int(m * extra) + 16, gen)
        lo, hi = torch.minimum(a, b), torch.maximum(a, b)
        fresh = ((lo << 32) | hi)[lo != hi]
        keys = torch.unique(torch.cat([keys, fresh]))
        if keys.numel() >= m or c["model"] == "ba":
            break
        extra = 0.5
    del a, b, lo, hi, fresh
    keys = keys[torch.randperm(keys.numel(), device=DEV, generator=gen)[:m]]
    names = torch.randperm(n, device=DEV, generator=gen).to(torch.int32)
    src, dst = names[keys >> 32], names[keys & 0xFFFFFFFF]
    vl = _labels(n, c["nvl"], c["zipf"], gen)
    el = _labels(src.numel(), c["nel"], c["zipf"], gen)
    return vl, src.contiguous(), dst.contiguous(), el


class _Walker:
    """Random walks over a graph's adjacency (both directions, sorted)."""

    def __init__(self, n, vl, src, dst, el):
        s, d = src.long(), dst.long()
        keys, at = torch.sort(torch.cat([(s << 32) | d, (d << 32) | s]))
        self.keys, self.el, self.vl = keys, torch.cat([el, el])[at].to(torch.int32), vl
        deg = torch.bincount(keys >> 32, minlength=n)
        self.first = torch.cumsum(deg, 0) - deg
        self.deg = deg
        self.starts = torch.nonzero(deg).flatten()

    def walks(self, count, steps, gen):
        """(vertices, edge labels) of `count` walks: host arrays (count, steps + 1) and (count, steps)."""
        v = self.starts[torch.randint(0, self.starts.numel(), (count,), device=DEV, generator=gen)]
        vs, ls = [v], []
        for _ in range(steps):
            x = torch.rand(count, device=DEV, generator=gen, dtype=torch.float64)
            e = self.first[v] + (x * self.deg[v]).long().clamp(max=self.deg[v] - 1)
            v = self.keys[e] & 0xFFFFFFFF
            vs.append(v)
            ls.append(self.el[e])
        return torch.stack(vs, 1).cpu().numpy(), torch.stack(ls, 1).cpu().numpy()

    def edge_labels(self, a, b):
        """Label of the edge of each pair, -1 where there is none (host arrays)."""
        k = (torch.from_numpy(a).to(DEV) << 32) | torch.from_numpy(b).to(DEV)
        at = torch.searchsorted(self.keys, k).clamp(max=self.keys.numel() - 1)
        return torch.where(self.keys[at] == k, self.el[at], -1).cpu().numpy()

    def labels(self, v):
        return self.vl[torch.from_numpy(v).to(DEV)].cpu().numpy()


class Query:
    """A query graph: vertices 0..k-1 with labels, labelled edges."""

    def __init__(self, k, vlabel, edges):
        self.k = k
        self.vlabel = np.ascontiguousarray(vlabel, dtype=np.uint32)
        e = np.array([(a, b, l) for (a, b), l in sorted(edges.items())], dtype=np.uint32).reshape(-1, 3)
        self.src, self.dst, self.elabel = (np.ascontiguousarray(e[:, i]) for i in range(3))


SHAPES = {"walk": ("walk",), "walk_cycle": ("walk_cycle",), "walk_dense": ("walk", "dense"),
          "mixed": ("tree", "walk_cycle", "dense")}


def _make_queries(w, specs, gen):
    """A query for each (k, shape): the first k vertices of a random walk with
    their labels and the walk's edges (walk), its first-visit edges (tree),
    one more edge among its vertices (walk_cycle) or all of them (dense).
    None where the walk met fewer than k vertices."""
    vs, ls = w.walks(len(specs), 8 * max(k for k, _ in specs), gen)
    seen, edges = [], []
    for i, (k, shape) in enumerate(specs):
        at, es = {int(vs[i, 0]): 0}, {}
        for t in range(ls.shape[1]):
            if len(at) == k:
                break
            a, b = int(vs[i, t]), int(vs[i, t + 1])
            new = b not in at
            x, y = at[a], at.setdefault(b, len(at))
            if new or shape != "tree":
                es[min(x, y), max(x, y)] = int(ls[i, t])
        seen.append(list(at) if len(at) == k else None)
        edges.append(es)
    pairs = [(i, x, y) for i, (k, shape) in enumerate(specs) if seen[i] and shape in ("walk_cycle", "dense")
             for x in range(k) for y in range(x + 1, k)]
    if pairs:
        a = np.array([seen[i][x] for i, x, _ in pairs], dtype=np.int64)
        b = np.array([seen[i][y] for i, _, y in pairs], dtype=np.int64)
        done = set()
        for (i, x, y), l in zip(pairs, w.edge_labels(a, b).tolist()):
            if l < 0 or (x, y) in edges[i] or i in done:
                continue
            edges[i][x, y] = l
            if specs[i][1] == "walk_cycle":
                done.add(i)
    lab = w.labels(np.array([v for s in seen if s for v in s], dtype=np.int64)) if any(seen) else None
    out, o = [], 0
    for (k, _), s, es in zip(specs, seen, edges):
        if s:
            out.append(Query(k, lab[o:o + k], es))
            o += k
        else:
            out.append(None)
    return out


def _fits(dg, q, cap, homo=False):
    """Whether no table of the query has more than `cap` rows."""
    flags = gsi.GSI_COUNT_ONLY | gsi.GSI_NO_FUSED | (gsi.GSI_HOMOMORPHISM if homo else 0)
    try:
        dg.query(q, flags=flags, max_rows=cap).free()
    except gsi.GsiError as e:
        if e.status not in (gsi.GSI_E_CAPACITY, gsi.GSI_E_NOMEM):
            raise
        return False
    return True


def _queries(c, w, dg, count, gen):
    """`count` queries of the case within its row limit."""
    rnd = np.random.default_rng([int(torch.randint(0, 1 << 31, (1,), device=DEV, generator=gen)), 7])
    out, tries = [], 0
    while len(out) < count:
        short = tries // 4  # shorter queries when the drawn ones are refused over and over
        specs = []
        for _ in range(max(8, count - len(out))):
            k = int(rnd.integers(c["kmin"], c["kmax"] + 1)) - short
            shape = SHAPES[c["shape"]]
            specs.append((max(2, k), shape[int(rnd.integers(0, len(shape)))]))
        for q in _make_queries(w, specs, gen):
            if q is not None and len(out) < count and (q.k == 2 or _fits(dg, q, c["cap"], c.get("homo", False))):
                out.append(q)
        tries += 1
    return out


_homes = collections.OrderedDict()  # graphs and contexts in use, least recent first


def _home(key, nbytes, make):
    """The thing kept under `key`, made when it is not there; the least
    recently used ones go when the arenas would pass 130 GB together."""
    if key not in _homes:
        while _homes and nbytes + sum(h.nbytes for h in _homes.values()) > 130 << 30:
            _homes.popitem(last=False)
        torch.cuda.empty_cache()
        _homes[key] = make()
        _homes[key].nbytes = nbytes
    _homes.move_to_end(key)
    return _homes[key]


class _Home:
    """A context over an arena of `nbytes`."""

    def __init__(self, nbytes):
        self.ctx = gsi.Context(nbytes)

    def __del__(self):
        if hasattr(self, "ctx"):
            self.ctx.close()


class _Resident(_Home):
    """A loaded graph, and a walker over it."""

    def __init__(self, c, nbytes):
        super().__init__(nbytes)
        vl, src, dst, el = _edges(c, _gen(19))
        self.dg = self.ctx.load_device(c["n"], vl, src, dst, el)
        self.walker = _Walker(c["n"], vl, src, dst, el)


def _graph(c):
    key = tuple(c[x] for x in ("model", "n", "m", "nvl", "nel", "zipf"))
    nbytes = gsi.gsi_graph_bytes_needed(c["n"], c["m"]) + (32 << 30)
    return _home(key, nbytes, lambda: _Resident(c, nbytes))


# ------------------------------------------------------------ multi-labels
class MultiQuery:
    def __init__(self, sets, edges):
        self.k = len(sets)
        self.qoff = np.cumsum([0] + [len(s) for s in sets]).astype(np.uint32)
        self.qlab = np.array([x for s in sets for x in s], dtype=np.uint32)
        e = np.array(sorted(edges), dtype=np.uint32).reshape(-1, 3)
        self.src, self.dst, self.elabel = (np.ascontiguousarray(e[:, i]) for i in range(3))


class _MultiGraph(_Home):
    """Vertices with 1 to 3 labels, pairs with 1 or 2 (one entry per label)."""

    def __init__(self, c, nbytes):
        super().__init__(nbytes)
        r = np.random.default_rng([19, c["n"]])
        n = self.n = c["n"]
        key = np.unique(r.integers(0, n, c["m"]).astype(np.int64) << 32 | r.integers(0, n, c["m"]))
        a, b = key >> 32, key & 0xFFFFFFFF
        key = np.unique(np.minimum(a, b)[a != b] << 32 | np.maximum(a, b)[a != b])
        a, b = key >> 32, key & 0xFFFFFFFF
        l = r.integers(0, c["nel"], a.shape[0])
        two = np.nonzero(r.random(a.shape[0]) < 0.25)[0]
        a, b = np.concatenate([a, a[two]]), np.concatenate([b, b[two]])
        l = np.concatenate([l, (l[two] + 1) % c["nel"]])
        self.src, self.dst, self.elabel = (x.astype(np.uint32) for x in (a, b, l))
        per = r.integers(1, 4, n)
        self.voff = np.concatenate([[0], np.cumsum(per)]).astype(np.uint64)
        start = np.repeat(r.integers(0, c["nvl"], n), per)
        self.vlab = ((start + 3 * (np.arange(start.shape[0]) - np.repeat(self.voff[:-1].astype(np.int64), per)))
                     % c["nvl"]).astype(np.uint32)
        order = np.argsort(np.concatenate([a, b]), kind="stable")
        self.nb, self.nl = np.concatenate([b, a])[order], np.concatenate([l, l])[order]
        self.first = np.concatenate([[0], np.cumsum(np.bincount(np.concatenate([a, b]), minlength=n))])
        self.dg = self.ctx.load_multi(self)

    def query(self, k, r):
        v = int(r.integers(0, self.n))
        at, edges = {v: 0}, set()
        for _ in range(8 * k):
            if len(at) == k or self.first[v] == self.first[v + 1]:
                break
            e = int(r.integers(self.first[v], self.first[v + 1]))
            w = int(self.nb[e])
            x, y = at[v], at.setdefault(w, len(at))
            edges.add((min(x, y), max(x, y), int(self.nl[e])))
            v = w
        if len(at) < k:
            return None
        sets = []
        for x in at:
            ls = self.vlab[int(self.voff[x]):int(self.voff[x + 1])].tolist()
            sets.append(sorted(ls[:int(r.integers(1, len(ls) + 1))]))
        return MultiQuery(sets, edges)

    def fits(self, q, cap):
        try:
            self.dg.query_multi(q, flags=gsi.GSI_COUNT_ONLY | gsi.GSI_NO_FUSED, max_rows=cap).free()
        except gsi.GsiError as e:
            if e.status not in (gsi.GSI_E_CAPACITY, gsi.GSI_E_NOMEM):
                raise
            return False
        return True


def _multi_graph(c):
    nbytes = gsi.gsi_graph_bytes_needed(c["n"], 2 * c["m"]) + (8 << 30)
    return _home(tuple(c[x] for x in ("n", "m", "nvl", "nel")), nbytes, lambda: _MultiGraph(c, nbytes))


# ------------------------------------------------------------------ passes
class State:
    """What the program holds between passes, and its last results."""

    def __init__(self, c):
        self.c, self.open, self.server = c, [], None

    def close(self):
        for r in self.open:
            r.free()
        self.open = []

    def __del__(self):
        if self.home.ctx.h:
            self.close()
            if self.server is not None:
                self.server.free()


def _load_home(c):
    """The context that graphs of the case's size are loaded into."""
    nbytes = gsi.gsi_graph_bytes_needed(c["n"], c["m"]) + (4 << 30)
    return _home((c["n"], c["m"]), nbytes, lambda: _Home(nbytes))


def prepare(case, seed):
    c, s, gen = case, State(case), _gen(1000 + seed)
    if c["kind"] == "load":
        s.home = _load_home(c)
        s.arrays = _edges(c, gen)
        dg = s.home.ctx.load_device(c["n"], *s.arrays)
        s.queries = _queries(c, _Walker(c["n"], *s.arrays), dg, 1, gen)
        dg.free()
    elif c["kind"] == "multi":
        s.home = _multi_graph(c)
        r, s.queries = np.random.default_rng([seed, 3]), []
        while len(s.queries) < c["nq"]:
            q = s.home.query(int(r.integers(c["kmin"], c["kmax"] + 1)), r)
            if q is not None and s.home.fits(q, c["cap"]):
                s.queries.append(q)
    else:
        s.home = _graph(c)
        s.queries = _queries(c, s.home.walker, s.home.dg, c["nq"], gen)
        if c["kind"] == "serve":
            s.server = s.home.dg.server(flags=gsi.GSI_COUNT_ONLY)
    if c["kind"] == "multi" or not c.get("count_only", True):
        words = c["nq"] * c["cap"] * c["kmax"]
        s.rows = (np.zeros(words, dtype=np.int32) if c["kind"] == "batch" else
                  torch.zeros(words, dtype=torch.int32, device=DEV))
    return s


def _keep_rows(s):
    """Every result's rows, one after the other, in the program's own device
    buffer (the rest of it stays zero)."""
    arena, at = s.home.ctx.arena, 0
    for r in s.open:
        n = r.count * r.k
        if n:
            p = gsi.gsi_result_device_rows(r.h) - arena.data_ptr()
            s.rows[at:at + n].copy_(arena[p:p + 4 * n].view(torch.int32))
            at += n
    return s.rows


def _numbers(counts, digests):
    return {"counts": np.array(counts, dtype=np.uint64).view(np.int64),
            "digests": np.array(digests, dtype=np.uint64).reshape(-1, 2).view(np.int64)}


def run(s):
    c, kind = s.c, s.c["kind"]
    s.close()
    if kind == "load":
        dg = s.home.ctx.load_device(c["n"], *s.arrays)
        r = dg.query(s.queries[0], flags=gsi.GSI_COUNT_ONLY)
        info = dg.info()
        out = _numbers([r.count], [r.digest])
        out["shape"] = np.array([info[x] for x in ("n_vertices", "n_edges", "n_edge_labels", "total_groups",
                                                   "max_chain")], dtype=np.int64)
        out["edges"] = np.array([gsi.gsi_graph_label_edges(dg.h, l) for l in range(c["nel"])], dtype=np.int64)
        r.free()
        dg.free()
        return out
    dg = s.home.dg
    if kind == "multi":
        s.open = [dg.query_multi(q, flags=gsi.GSI_NO_CHUNKS) for q in s.queries]
        return {**_numbers([r.count for r in s.open], [r.digest for r in s.open]),
                "rows": _keep_rows(s)}
    if kind == "single":
        flags = ((gsi.GSI_COUNT_ONLY if c["count_only"] else 0) | (0 if c["chunks"] else gsi.GSI_NO_CHUNKS) |
                 (gsi.GSI_HOMOMORPHISM if c["homo"] else 0))
        s.open = [dg.query(q, flags=flags) for q in s.queries]
        out = _numbers([r.count for r in s.open], [r.digest for r in s.open])
        if not c["count_only"]:
            out["rows"] = _keep_rows(s)
        return out
    if kind == "batch":
        b = dg.batch(s.queries, flags=gsi.GSI_COUNT_ONLY if c["count_only"] else 0)
        out = _numbers(*b.results())
        if not c["count_only"]:
            at = 0
            for i in range(len(s.queries)):
                r = b.rows(i).view(np.int32).ravel()
                s.rows[at:at + r.size] = r
                at += r.size
            out["rows"] = s.rows
        b.free()
        return out
    tickets, done = [s.server.submit(q) for q in s.queries], 0
    while done < len(tickets):
        s.server.step()
        done += len(s.server.poll())
    answers = [s.server.answer(t) for t in tickets]
    for t in tickets:
        s.server.release(t)
    return _numbers([a["count"] for a in answers], [a["digest"] for a in answers])


def work(case):
    """Bytes a pass cannot do without: a query tests every vertex's label
    once (4 bytes each) and, where rows are written, writes them (their
    number depends on the seed: a tenth of the row limit is taken); a load
    reads its arrays and writes the lists (two directions) and the
    signatures (64 bytes a vertex)."""
    c = case
    if c["kind"] == "load":
        return {"bytes": 4.0 * c["n"] + 12.0 * c["m"] + 8.0 * c["m"] + 64.0 * c["n"], "flops": 0.0}
    rows = 0.0
    if c["kind"] == "single" and not c["count_only"]:
        rows = 4.0 * c["kmax"] * min(c["cap"] / 10, c["n"])
    return {"bytes": c["nq"] * (4.0 * c["n"] + rows), "flops": 0.0}


def exact(case, seed):
    """Every output is a whole number (vertex ids, counts, digests), which
    has to be equal: there is no 64-bit value to be near to."""
    return None
