// Device build of the data-graph structures a query needs:
//   * PCSR(G,l) for every edge label l (Sec. IV, Definition 4, Algorithm 1);
//   * the column-first vertex signature table (Sec. III-A).
//
// Layout choices (the paper leaves the hash and overflow placement open):
//   * both directions of every edge are stored, each vertex's l-neighbours
//     ascending;
//   * label l owns |V(D_l)| groups of 16 (vertex, offset) pairs (128 bytes);
//     v's home group is pcsr_home(v, H_l) with H_l = |V(D_l)|;
//   * a group keeps its 15 smallest home keys; further keys go 15 per group
//     to empty groups of the same label, taken in ascending index order and
//     handed to overflowing groups in ascending home index, linked through
//     the GID of pair 15 (0xFFFFFFFF ends a chain).  Claim 1 of the paper
//     guarantees enough empty groups;
//   * ci is written in group order then slot order; an unused slot holds
//     (0xFFFFFFFF, END), so the list in slot s ends at the offset of pair s+1.
//
// Pipeline: check the edges -> directed entries sorted by (src, dst), whose
// vertices' entries are contiguous: signatures -> one more stable pass on the
// label: (label, src, dst) order -> runs of equal (label, src) are the keys
// of the partitions -> home groups -> stable sort of keys by group -> chains
// -> group sizes -> scan -> write groups and scatter neighbour lists.
#include <algorithm>
#include <chrono>
#include <cstring>

#include "gsi_internal.h"

namespace gsi {

constexpr uint32_t BT = 256;

static uint32_t blocks(uint64_t n, uint64_t per = BT) {
    uint64_t b = (n + per - 1) / per;
    if (b == 0) b = 1;
    if (b > 0x7FFFFFFFull) fail(GSI_E_INVALID, "grid too large");
    return (uint32_t)b;
}

static int bits_for(uint64_t maxval) {
    int b = 0;
    while (b < 64 && (maxval >> b) != 0) b++;
    return b;
}

enum : uint32_t { ERR_RANGE = 1, ERR_SELF = 2, ERR_LABEL = 4, ERR_DUP = 8, ERR_CLAIM1 = 16 };

// range, self-loop and label checks; the largest label of each workgroup's
// edges (no same-address atomics)
__global__ __launch_bounds__(BT) void k_validate(const uint32_t *src, const uint32_t *dst, const uint32_t *el,
                                                 uint64_t m, uint32_t n, uint32_t *err, uint32_t *maxlab_part) {
    uint32_t f = 0, mx = 0;
    for (uint64_t e = (uint64_t)blockIdx.x * BT + threadIdx.x; e < m; e += (uint64_t)gridDim.x * BT) {
        const uint32_t a = src[e], b = dst[e], l = el[e];
        if (a >= n || b >= n) f |= ERR_RANGE;
        if (a == b) f |= ERR_SELF;
        if (l >= GSI_MAX_EDGE_LABELS) f |= ERR_LABEL;
        mx = l > mx ? l : mx;
    }
    if (f) atomicOr(err, f);
    __shared__ uint32_t s_max[BT / 64];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        uint32_t t = __shfl_xor(mx, o, 64);
        mx = t > mx ? t : mx;
    }
    if (lane_id() == 0) s_max[threadIdx.x >> 6] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
        mx = 0;
#pragma unroll
        for (int q = 0; q < BT / 64; q++) mx = s_max[q] > mx ? s_max[q] : mx;
        maxlab_part[blockIdx.x] = mx;
    }
}

// both directions of every edge as three arrays (graphs whose entries do
// not pack into 64 bits)
__global__ __launch_bounds__(BT) void k_expand(const uint32_t *src, const uint32_t *dst, const uint32_t *el,
                                               uint64_t m, uint32_t *os, uint32_t *od, uint32_t *ol) {
    const uint64_t e = (uint64_t)blockIdx.x * BT + threadIdx.x;
    if (e >= m) return;
    const uint32_t a = src[e], b = dst[e], l = el[e];
    os[2 * e] = a;
    od[2 * e] = b;
    ol[2 * e] = l;
    os[2 * e + 1] = b;
    od[2 * e + 1] = a;
    ol[2 * e + 1] = l;
}

// The sorted directed entries: packed keys (label, source, destination;
// vb bits an end) or, with key null, three arrays.
struct Entries {
    const uint64_t *key;
    const uint32_t *s, *d, *l;
    int vb;
};
struct Entry {
    uint32_t s, d, l;
};
__device__ __forceinline__ Entry entry_at(const Entries &E, uint64_t p) {
    if (E.key) {
        const uint64_t k = E.key[p];
        const uint32_t mask = (uint32_t)((1ull << E.vb) - 1);
        return {(uint32_t)(k >> E.vb) & mask, (uint32_t)k & mask, (uint32_t)(k >> (2 * E.vb))};
    }
    return {E.s[p], E.d[p], E.l[p]};
}

__global__ __launch_bounds__(1024) void k_max_u32(const uint32_t *part, uint64_t n, uint32_t *out) {
    __shared__ uint32_t s_m[16];
    uint32_t mx = 0;
    for (uint64_t i = threadIdx.x; i < n; i += 1024) mx = part[i] > mx ? part[i] : mx;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        uint32_t t = __shfl_xor(mx, o, 64);
        mx = t > mx ? t : mx;
    }
    if (lane_id() == 0) s_m[threadIdx.x >> 6] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int q = 0; q < 16; q++) mx = s_m[q] > mx ? s_m[q] : mx;
        *out = mx;
    }
}

// multi-labelled graphs, after sorting by (label, src, dst): equal
// neighbours with equal labels are the same labelled edge given twice
__global__ __launch_bounds__(BT) void k_check_dup_labelled(Entries E, uint64_t nd, uint32_t *err) {
    const uint64_t p = (uint64_t)blockIdx.x * BT + threadIdx.x;
    if (p == 0 || p >= nd) return;
    const Entry x = entry_at(E, p), y = entry_at(E, p - 1);
    if (x.s == y.s && x.d == y.d && x.l == y.l) atomicOr(err, (uint32_t)ERR_DUP);
}

// Runs of equal (label, src) in the (label, src, dst)-sorted entries.  A
// workgroup takes RUN_TILE consecutive entries, RUN_ITEMS rounds of one per
// thread; the run of entry p is the number of run heads at or before it,
// less one: the heads before the tile (scanned tile counts), before the
// wave's round (LDS) and before the lane (ballot).  No array of the entries'
// size is written for it.
constexpr uint32_t RUN_ITEMS = 8, RUN_TILE = BT * RUN_ITEMS;

__device__ __forceinline__ bool run_head(const Entries &E, uint64_t p, const Entry &x, bool *newlab) {
    if (p == 0) {
        *newlab = true;
        return true;
    }
    const Entry y = entry_at(E, p - 1);
    *newlab = x.l != y.l;
    return *newlab || x.s != y.s;
}

__global__ __launch_bounds__(BT) void k_count_runs(Entries E, uint64_t nd, uint32_t *cnt) {
    __shared__ uint32_t s_c[BT / 64];
    const uint64_t base = (uint64_t)blockIdx.x * RUN_TILE;
    uint32_t c = 0;
#pragma unroll
    for (uint32_t i = 0; i < RUN_ITEMS; i++) {
        const uint64_t p = base + i * BT + threadIdx.x;
        const uint64_t pp = p < nd ? p : nd - 1;
        bool nl;
        const bool h = run_head(E, pp, entry_at(E, pp), &nl) && p < nd;
        c += (uint32_t)__popcll(__ballot(h));
    }
    if (lane_id() == 0) s_c[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t t = 0;
#pragma unroll
        for (uint32_t q = 0; q < BT / 64; q++) t += s_c[q];
        cnt[blockIdx.x] = t;
    }
}

// the runs of the thread's RUN_ITEMS entries (r[i]; garbage past nd), and
// whether each is its run's head and its label's first
struct TileRuns {
    uint64_t r[RUN_ITEMS];
    Entry x[RUN_ITEMS];
    bool head[RUN_ITEMS], newlab[RUN_ITEMS];
};
__device__ __forceinline__ void tile_runs(const Entries &E, uint64_t nd, const uint64_t *off, TileRuns &t) {
    __shared__ uint32_t s_c[RUN_ITEMS * (BT / 64)];
    const uint64_t base = (uint64_t)blockIdx.x * RUN_TILE;
    const uint32_t w = threadIdx.x >> 6;
    uint32_t upto[RUN_ITEMS];  // heads of the wave's round at or before the lane
#pragma unroll
    for (uint32_t i = 0; i < RUN_ITEMS; i++) {
        const uint64_t p = base + i * BT + threadIdx.x;
        const uint64_t pp = p < nd ? p : nd - 1;
        t.x[i] = entry_at(E, pp);
        t.head[i] = run_head(E, pp, t.x[i], &t.newlab[i]) && p < nd;
        const uint64_t mask = __ballot(t.head[i]);
        upto[i] = rank_below(mask) + (t.head[i] ? 1u : 0u);
        if (lane_id() == 0) s_c[i * (BT / 64) + w] = (uint32_t)__popcll(mask);
    }
    __syncthreads();
    if (threadIdx.x < 64) {
        const uint32_t c = threadIdx.x < RUN_ITEMS * (BT / 64) ? s_c[threadIdx.x] : 0u;
        const uint32_t inc = wave_inclusive_sum(c);
        if (threadIdx.x < RUN_ITEMS * (BT / 64)) s_c[threadIdx.x] = inc - c;
    }
    __syncthreads();
    const uint64_t first = off[blockIdx.x];
#pragma unroll
    for (uint32_t i = 0; i < RUN_ITEMS; i++) t.r[i] = first + s_c[i * (BT / 64) + w] + upto[i] - 1;
}

// label segments: first entry, end, first run and end of runs
struct Segments {
    uint64_t *lo, *hi, *rb, *re;
};

// run r = (label, vertex) with its first entry, and the label segments
__global__ __launch_bounds__(BT) void k_runs(Entries E, uint64_t nd, const uint64_t *off, uint32_t *run_start,
                                             uint32_t *run_vid, uint32_t *run_lab, Segments seg) {
    TileRuns t;
    tile_runs(E, nd, off, t);
#pragma unroll
    for (uint32_t i = 0; i < RUN_ITEMS; i++) {
        const uint64_t p = (uint64_t)blockIdx.x * RUN_TILE + i * BT + threadIdx.x;
        if (p >= nd) continue;
        const uint32_t l = t.x[i].l;
        if (t.head[i]) {
            run_start[t.r[i]] = (uint32_t)p;
            run_vid[t.r[i]] = t.x[i].s;
            run_lab[t.r[i]] = l;
        }
        if (t.newlab[i]) {
            seg.lo[l] = p;
            seg.rb[l] = t.r[i];
            if (p) {
                const uint32_t lp = entry_at(E, p - 1).l;
                seg.hi[lp] = p;
                seg.re[lp] = t.r[i];
            }
        }
        if (p + 1 == nd) {
            seg.hi[l] = nd;
            seg.re[l] = t.r[i] + 1;
        }
    }
}

struct LabelTab {
    const uint64_t *rb;   // first global group of label
    const uint32_t *G;    // groups of label
    const uint32_t *H;    // home groups of label
    const uint64_t *seg;  // first directed entry (= first ci entry) of label
};

// home group of every run, above the run's number in a 64-bit sort key
__global__ void k_home(const uint32_t *run_vid, const uint32_t *run_lab, uint64_t R, LabelTab t, uint64_t *key,
                       uint32_t *cnt) {
    uint64_t r = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= R) return;
    uint32_t l = run_lab[r];
    uint32_t g = (uint32_t)t.rb[l] + pcsr_home(run_vid[r], t.H[l]);
    key[r] = ((uint64_t)g << 32) | r;
    atomicAdd(&cnt[g], 1u);
}

// label of a global group: the last label whose first group is <= grp
// (labels without groups carry the first group of the next label, so the
// search lands on the label that owns grp)
__device__ __forceinline__ uint32_t label_of_group(const uint64_t *rb, uint32_t nlab, uint64_t grp) {
    uint32_t lo = 0, hi = nlab - 1;
    while (lo < hi) {
        uint32_t mid = (lo + hi + 1) >> 1;
        if (rb[mid] <= grp) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

__global__ void k_overflow_flags(const uint32_t *cnt, uint64_t R, uint32_t *need, uint32_t *empty) {
    uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= R) return;
    uint32_t c = cnt[g];
    need[g] = c > KEYS_PER_GROUP ? (c - KEYS_PER_GROUP + KEYS_PER_GROUP - 1) / KEYS_PER_GROUP : 0u;
    empty[g] = c == 0 ? 1u : 0u;
}

// the e-th empty group (ascending) of each label, label-relative ids
__global__ void k_empty_list(const uint32_t *empty, const uint64_t *escan, uint64_t R, const uint64_t *rb,
                             const uint32_t *G, uint32_t nlab, uint32_t *elist) {
    uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= R || !empty[g]) return;
    uint32_t l = label_of_group(rb, nlab, g);
    uint64_t base = rb[l];
    uint64_t at = base + (escan[g] - escan[base]);
    if (at < R) elist[at] = (uint32_t)(g - base);
}

__global__ void k_claim1(const uint64_t *nscan, const uint64_t *escan, const uint64_t *rb, const uint32_t *G,
                         uint32_t nlab, uint32_t *err) {
    uint32_t l = blockIdx.x * blockDim.x + threadIdx.x;
    if (l >= nlab || G[l] == 0) return;
    uint64_t a = rb[l], b = a + G[l];
    if (nscan[b] - nscan[a] > escan[b] - escan[a]) atomicOr(err, (uint32_t)ERR_CLAIM1);
}

// chain every overflowing group through its empty groups
__global__ void k_chains(const uint32_t *need, const uint64_t *nscan, const uint32_t *elist, uint64_t R,
                         const uint64_t *rb, const uint32_t *G, uint32_t nlab, uint32_t *next, uint32_t *owner,
                         uint32_t *chain_idx, uint32_t *max_chain) {
    uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= R || need[g] == 0) return;
    uint32_t l = label_of_group(rb, nlab, g);
    uint64_t base = rb[l];
    uint64_t first = nscan[g] - nscan[base];
    uint64_t prev = g;
    if (base + first + need[g] > base + G[l]) return;  // Claim 1 violated: reported by k_claim1
    for (uint32_t m = 1; m <= need[g]; m++) {
        uint32_t e = elist[base + first + m - 1];
        if (e >= G[l]) return;  // never reached when Claim 1 holds
        next[prev] = e;
        owner[base + e] = (uint32_t)(g - base);
        chain_idx[base + e] = m;
        prev = base + e;
    }
    atomicMax(max_chain, need[g] + 1);
}

// keys held by each group and the total length of their lists
__global__ void k_group_keys(const uint32_t *cnt, const uint64_t *gstart, const uint32_t *owner,
                             const uint32_t *chain_idx, const uint64_t *sorted, const uint32_t *run_start,
                             uint64_t R, uint64_t nd, const uint64_t *rb, const uint32_t *G, uint32_t nlab,
                             uint64_t *kfirst, uint32_t *nkeys, uint32_t *gdeg) {
    uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= R) return;
    uint64_t first = 0;
    uint32_t nk = 0;
    uint32_t c = cnt[g];
    if (c > 0) {
        first = gstart[g];
        nk = c < KEYS_PER_GROUP ? c : KEYS_PER_GROUP;
    } else if (owner[g] != NONE32) {
        uint32_t l = label_of_group(rb, nlab, g);
        uint64_t h = rb[l] + owner[g];
        uint32_t mi = chain_idx[g];
        first = gstart[h] + (uint64_t)KEYS_PER_GROUP * mi;
        uint32_t left = cnt[h] - KEYS_PER_GROUP * mi;
        nk = left < KEYS_PER_GROUP ? left : KEYS_PER_GROUP;
    }
    uint32_t deg = 0;
    for (uint32_t s = 0; s < nk; s++) {
        uint32_t r = (uint32_t)sorted[first + s];
        uint64_t end = (r + 1 < R) ? run_start[r + 1] : nd;
        deg += (uint32_t)(end - run_start[r]);
    }
    kfirst[g] = first;
    nkeys[g] = nk;
    gdeg[g] = deg;
}

// write the 16 pairs of each group; remember each key's list offset
__global__ void k_write_groups(const uint64_t *kfirst, const uint32_t *nkeys, const uint64_t *gci,
                               const uint32_t *next, const uint64_t *sorted, const uint32_t *run_start,
                               const uint32_t *run_vid, uint64_t R, uint64_t nd, const uint64_t *rb,
                               const uint32_t *G, const uint64_t *seg, uint32_t nlab, uint32_t *gl,
                               uint32_t *run_off) {
    uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= R) return;
    uint32_t l = label_of_group(rb, nlab, g);
    uint64_t lb = seg[l];
    uint32_t pos = (uint32_t)(gci[g] - lb);
    uint32_t end = (uint32_t)(gci[g + 1] - lb);
    uint32_t pr[GROUP_WORDS];
    uint32_t nk = nkeys[g];
    uint64_t first = kfirst[g];
#pragma unroll
    for (uint32_t s = 0; s < KEYS_PER_GROUP; s++) {
        if (s < nk) {
            uint32_t r = (uint32_t)sorted[first + s];
            uint64_t e = (r + 1 < R) ? run_start[r + 1] : nd;
            pr[2 * s] = run_vid[r];
            pr[2 * s + 1] = pos;
            run_off[r] = pos;
            pos += (uint32_t)(e - run_start[r]);
        } else {
            pr[2 * s] = NONE32;
            pr[2 * s + 1] = end;
        }
    }
    pr[2 * KEYS_PER_GROUP] = next[g];
    pr[2 * KEYS_PER_GROUP + 1] = end;
    uint4 *dstv = reinterpret_cast<uint4 *>(gl + g * GROUP_WORDS);
#pragma unroll
    for (int i = 0; i < 8; i++) dstv[i] = make_uint4(pr[4 * i], pr[4 * i + 1], pr[4 * i + 2], pr[4 * i + 3]);
}

__global__ __launch_bounds__(BT) void k_scatter_ci(Entries E, uint64_t nd, const uint64_t *off,
                                                   const uint32_t *run_start, const uint32_t *run_off,
                                                   const uint64_t *seg, uint32_t *ci) {
    TileRuns t;
    tile_runs(E, nd, off, t);
#pragma unroll
    for (uint32_t i = 0; i < RUN_ITEMS; i++) {
        const uint64_t p = (uint64_t)blockIdx.x * RUN_TILE + i * BT + threadIdx.x;
        if (p >= nd) continue;
        const uint64_t r = t.r[i];
        const uint64_t at = seg[t.x[i].l] + run_off[r] + (uint32_t)(p - run_start[r]);
        if (at < nd) ci[at] = t.x[i].d;
    }
}

// Signatures (Sec. III-A): word 0 = label; each directed entry (v -> w, l)
// adds the pair (l, L_V(w)) to v's two-bit group: the first pair sets the
// low bit (01); any later pair finds it set and raises the high bit (11).
__global__ void k_sig_labels(const uint32_t *vl, uint32_t n, uint32_t *sig) {
    uint64_t v = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    sig[v] = vl[v];
#pragma unroll
    for (int w = 1; w < GSI_SIG_WORDS; w++) sig[(uint64_t)w * n + v] = 0;
}

// Multi-labelled vertices (Sec. VII-B): word 0 holds every label of v
// hashed to one of its 32 bits, so the filter tests containment there and a
// refinement pass checks the label sets exactly.
__global__ void k_sig_labels_multi(const uint32_t *off, const uint32_t *lab, uint32_t n, uint32_t *sig) {
    uint64_t v = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    uint32_t b = 0;
    for (uint32_t t = off[v]; t < off[v + 1]; t++) b |= label_bit(lab[t]);
    sig[v] = b;
#pragma unroll
    for (int w = 1; w < GSI_SIG_WORDS; w++) sig[(uint64_t)w * n + v] = 0;
}

// every directed entry (v -> w, l) adds the pair (l, x) for each label x of w
__global__ __launch_bounds__(BT) void k_sig_pairs_multi(Entries E, const uint32_t *off, const uint32_t *lab,
                                                        uint64_t nd, uint32_t n, uint32_t *sig) {
    const uint64_t p = (uint64_t)blockIdx.x * BT + threadIdx.x;
    if (p >= nd) return;
    const Entry x = entry_at(E, p);
    for (uint32_t t = off[x.d]; t < off[x.d + 1]; t++) {
        uint32_t g = sig_group(x.l, lab[t]);
        uint32_t *word = sig + (uint64_t)(1 + g / 16) * n + x.s;
        uint32_t lo = 1u << (2 * (g % 16));
        uint32_t old = atomicOr(word, lo);
        if (old & lo) atomicOr(word, lo << 1);
    }
}

// Signatures of a single-label graph from the (src, dst)-sorted entries,
// words 1..15 zero on entry; also flags repeated vertex pairs (equal
// neighbours).  A workgroup takes SIG_TILE consecutive entries, whose
// vertices are consecutive: their words are gathered in LDS, SIG_SPAN
// vertices at a time, and written column by column; only the tile's first
// and last vertex, which other tiles may hold entries of too, are merged
// with atomics.  Two atomics per entry on the table itself took 14.8 ms for
// 2*10^8 entries; this takes 3.9 ms, bound by the gather of the neighbours'
// labels.
constexpr uint32_t SIG_ITEMS = 16, SIG_TILE = BT * SIG_ITEMS, SIG_SPAN = BT;

__global__ __launch_bounds__(BT) void k_signatures(Entries E, const uint32_t *vl, uint64_t nd, uint32_t n,
                                                   uint32_t *sig, uint32_t *err) {
    __shared__ uint32_t s_sig[GSI_SIG_WORDS - 1][SIG_SPAN];
    __shared__ uint32_t s_next[BT / 64];
    const uint64_t base = (uint64_t)blockIdx.x * SIG_TILE;
    const uint64_t end = base + SIG_TILE < nd ? base + SIG_TILE : nd;
    uint32_t v[SIG_ITEMS];
    uint32_t w[SIG_ITEMS];  // destination, then its label, then the group
    uint32_t el[SIG_ITEMS];
    bool dup = false;
#pragma unroll
    for (uint32_t i = 0; i < SIG_ITEMS; i++) {
        const uint64_t p = base + i * BT + threadIdx.x;
        const uint64_t pp = p < end ? p : end - 1;
        const Entry x = entry_at(E, pp), y = entry_at(E, pp ? pp - 1 : 0);
        dup |= p < end && p > 0 && x.s == y.s && x.d == y.d;
        v[i] = x.s;
        w[i] = x.d;
        el[i] = x.l;
    }
#pragma unroll
    for (uint32_t i = 0; i < SIG_ITEMS; i++) w[i] = vl[w[i]];
#pragma unroll
    for (uint32_t i = 0; i < SIG_ITEMS; i++) {
        w[i] = sig_group(el[i], w[i]);
        if (base + i * BT + threadIdx.x >= end) v[i] = NONE32;  // no vertex
    }
    if (dup) atomicOr(err, (uint32_t)ERR_DUP);
    const uint32_t first = __builtin_amdgcn_readfirstlane(entry_at(E, base).s);
    const uint32_t last = __builtin_amdgcn_readfirstlane(entry_at(E, end - 1).s);
    const bool left = base > 0 && entry_at(E, base - 1).s == first;
    const bool right = end < nd && entry_at(E, end).s == last;
    uint32_t v0 = first;
    for (;;) {
#pragma unroll
        for (uint32_t q = 0; q < GSI_SIG_WORDS - 1; q++) s_sig[q][threadIdx.x] = 0;
        __syncthreads();
        uint32_t next = NONE32;  // first vertex past the span
#pragma unroll
        for (uint32_t i = 0; i < SIG_ITEMS; i++) {
            if (v[i] < v0) continue;
            if (v[i] - v0 >= SIG_SPAN) {
                next = v[i] < next ? v[i] : next;
                continue;
            }
            uint32_t *word = &s_sig[w[i] / 16][v[i] - v0];
            const uint32_t lo = 1u << (2 * (w[i] % 16));
            // a hub's entries mostly meet full groups: look before the atomic
            if ((*word & (3 * lo)) == 3 * lo) continue;
            const uint32_t old = atomicOr(word, lo);
            if (old & lo) atomicOr(word, lo << 1);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const uint32_t t = __shfl_xor(next, o, 64);
            next = t < next ? t : next;
        }
        if (lane_id() == 0) s_next[threadIdx.x >> 6] = next;
        __syncthreads();
        const uint32_t vv = v0 + threadIdx.x;
        if (vv >= v0 && vv <= last) {
            const bool shared = (vv == first && left) || (vv == last && right);
#pragma unroll
            for (uint32_t q = 0; q < GSI_SIG_WORDS - 1; q++) {
                const uint32_t x = s_sig[q][threadIdx.x];
                if (x == 0) continue;
                uint32_t *word = sig + (uint64_t)(1 + q) * n + vv;
                if (!shared) {
                    *word = x;
                } else {
                    // a group that two tiles have an entry of holds two or more
                    const uint32_t both = atomicOr(word, x) & x & 0x55555555u;
                    if (both) atomicOr(word, both << 1);
                }
            }
        }
#pragma unroll
        for (uint32_t q = 0; q < BT / 64; q++) next = s_next[q] < next ? s_next[q] : next;
        next = __builtin_amdgcn_readfirstlane(next);
        if (next == NONE32) break;
        v0 = next;
        __syncthreads();
    }
}

void build_graph(gsi_graph *g, const uint32_t *vl, const uint32_t *src, const uint32_t *dst, const uint32_t *el) {
    gsi_ctx *c = g->ctx;
    auto t0 = std::chrono::steady_clock::now();
    const uint32_t n = g->n;
    const uint64_t m = g->m, nd = 2 * m;
    Scratch s(c);

    uint64_t *scal = s.get<uint64_t>(8, "scalars");
    fill_u64(c, scal, 0, 8);
    uint32_t *err = reinterpret_cast<uint32_t *>(scal);       // scal[0] low word
    uint32_t *maxlab = reinterpret_cast<uint32_t *>(scal + 1);
    uint32_t *maxchain = reinterpret_cast<uint32_t *>(scal + 2);

    // persistent signature table first (independent of everything else)
    g->sig = persist<uint32_t>(c, (uint64_t)GSI_SIG_WORDS * n, "signature table");
    // CI_PAD spare elements: searches read aligned windows that may pass a list's end
    g->ci = persist<uint32_t>(c, nd + CI_PAD, "ci");

    if (m) {
        const uint32_t nb = std::min<uint32_t>(blocks(m), 4096);
        uint32_t *mpart = s.get<uint32_t>(nb, "label maxima");
        launch(c, "k_validate", 12.0 * m, k_validate, nb, BT, src, dst, el, m, n, err, mpart);
        launch(c, "k_max_u32", 4.0 * nb, k_max_u32, 1, 1024, (const uint32_t *)mpart, (uint64_t)nb, maxlab);
    }
    uint64_t hs[3];
    read_scalars(c, scal, hs, 3);
    uint32_t e0 = (uint32_t)hs[0];
    if (e0 & ERR_RANGE) fail(GSI_E_INVALID, "edge endpoint out of range");
    if (e0 & ERR_SELF) fail(GSI_E_INVALID, "self-loop in data graph");
    if (e0 & ERR_LABEL) fail(GSI_E_INVALID, "edge label >= %u", (unsigned)GSI_MAX_EDGE_LABELS);
    uint32_t nlab = m ? (uint32_t)hs[1] + 1 : 0;
    g->nlab = nlab;

    if (g->multi)
        launch(c, "k_sig_labels", 8.0 * n + 64.0 * n, k_sig_labels_multi, blocks(n), BT, (const uint32_t *)g->vl_off,
               (const uint32_t *)g->vl_lab, n, g->sig);
    else
        launch(c, "k_sig_labels", 8.0 * n + 60.0 * n, k_sig_labels, blocks(n), BT, vl, n, g->sig);

    // (src, dst) order: signatures and the check for repeated pairs; then a
    // stable sort on the label.  Entries that pack into 64 bits (2 vb + lb;
    // 51 bits for 8.4M vertices and 20 labels) are sorted as keys, others
    // (more than 2^24 vertices, depending on the labels) as three arrays.
    const int vb = bits_for(n - 1 ? n - 1 : 1), lb = bits_for(nlab > 1 ? nlab - 1 : 0);
    Entries E{nullptr, nullptr, nullptr, nullptr, vb};
    auto by_vertex = [&]() {
        if (!g->multi)
            launch(c, "k_signatures", 12.0 * nd + 60.0 * n, k_signatures, blocks(nd, SIG_TILE), BT, E, vl, nd, n,
                   g->sig, err);
    };
    if (m && 2 * vb + std::max(lb, 1) <= 64) {
        uint64_t *ka = s.get<uint64_t>(nd, "sort keys"), *kb = s.get<uint64_t>(nd, "sort keys");
        if (edge_key_sort(c, (uint32_t)m, src, dst, el, vb, ka, kb, s)) std::swap(ka, kb);
        E.key = ka;
        by_vertex();
        if (key_sort(c, (uint32_t)nd, ka, kb, 2 * vb, 2 * vb + lb, s)) std::swap(ka, kb);
        E.key = ka;
        s.drop(kb);
    } else if (m) {
        uint32_t *A[3], *B[3];
        for (int i = 0; i < 3; i++) {
            A[i] = s.get<uint32_t>(nd, "sort buffer");
            B[i] = s.get<uint32_t>(nd, "sort buffer");
        }
        launch(c, "k_expand", 36.0 * m, k_expand, blocks(m), BT, src, dst, el, m, A[0], A[1], A[2]);
        std::vector<SortPass> passes;
        for (int sh = 0; sh < vb; sh += 8) passes.push_back({1, sh});
        for (int sh = 0; sh < vb; sh += 8) passes.push_back({0, sh});
        uint32_t **cur = A, **other = B;
        if (radix_sort(c, (uint32_t)nd, A, B, passes, s)) std::swap(cur, other);
        E.s = cur[0], E.d = cur[1], E.l = cur[2];
        by_vertex();
        std::vector<SortPass> lp;
        for (int sh = 0; sh < lb; sh += 8) lp.push_back({2, sh});
        if (radix_sort(c, (uint32_t)nd, cur, other, lp, s)) std::swap(cur, other);
        E.s = cur[0], E.d = cur[1], E.l = cur[2];
    }
    if (m && g->multi) {
        launch(c, "k_check_dup", 12.0 * nd, k_check_dup_labelled, blocks(nd), BT, E, nd, err);
        launch(c, "k_sig_pairs", 24.0 * nd, k_sig_pairs_multi, blocks(nd), BT, E, (const uint32_t *)g->vl_off,
               (const uint32_t *)g->vl_lab, nd, n, g->sig);
    }

    // runs and label segments
    const uint32_t nrt = blocks(nd, RUN_TILE);
    uint32_t *rcnt = s.get<uint32_t>(nrt, "run counts");
    uint64_t *roff = s.get<uint64_t>((uint64_t)nrt + 1, "run offsets");
    uint64_t R = 0;
    if (m) {
        launch(c, "k_count_runs", 8.0 * nd, k_count_runs, nrt, BT, E, nd, rcnt);
        exclusive_scan(c, rcnt, nrt, roff, s, scal + 3);
    }
    uint64_t hr[4];
    read_scalars(c, scal, hr, 4);
    R = hr[3];
    if ((uint32_t)hr[0] & ERR_DUP)
        fail(GSI_E_INVALID, g->multi ? "the same labelled edge is given twice in the data graph"
                                     : "repeated vertex pair (parallel edge) in data graph");
    g->total_groups = R;
    const bool keep_cr = (g->flags & GSI_GRAPH_KEEP_CR) != 0;
    uint32_t *run_start = keep_cr ? persist<uint32_t>(c, R ? R : 1, "cr starts") : s.get<uint32_t>(R, "run start");
    uint32_t *run_vid = keep_cr ? persist<uint32_t>(c, R ? R : 1, "cr vertices") : s.get<uint32_t>(R, "run vertex");
    if (keep_cr) {
        g->cr_start = run_start;
        g->cr_vid = run_vid;
    }
    uint32_t *run_lab = s.get<uint32_t>(R, "run label");
    // label table on the device: segments and runs as found, then (from the
    // host) first group, first entry, groups and home groups of each label
    uint64_t *seg = s.get<uint64_t>(4 * (uint64_t)nlab + 1, "label segments");
    const Segments sg{seg, seg + nlab, seg + 2 * (uint64_t)nlab, seg + 3 * (uint64_t)nlab};
    std::vector<uint64_t> hseg(4 * (uint64_t)nlab);
    if (m) {
        fill_u64(c, seg, 0, 4 * (uint64_t)nlab);
        launch(c, "k_runs", 8.0 * nd + 12.0 * R, k_runs, nrt, BT, E, nd, (const uint64_t *)roff, run_start, run_vid,
               run_lab, sg);
        GSI_HIP(hipMemcpyAsync(hseg.data(), seg, 32ull * nlab, hipMemcpyDeviceToHost, c->stream));
        sync(c);
    }
    const uint64_t *h_lo = hseg.data(), *h_hi = h_lo + nlab, *h_rb = h_hi + nlab, *h_re = h_rb + nlab;
    g->group_base.assign(nlab, 0);
    g->G.assign(nlab, 0);
    g->H.assign(nlab, 0);
    g->ci_base.assign(nlab, 0);
    g->edges.assign(nlab, 0);
    // empty labels get the start of the next non-empty label so that group
    // ranges stay sorted for the label-of-group search
    uint64_t nextb = R;
    for (int64_t l = (int64_t)nlab - 1; l >= 0; l--) {
        if (h_re[l] > h_rb[l]) {
            g->group_base[l] = h_rb[l];
            g->G[l] = (uint32_t)(h_re[l] - h_rb[l]);
            g->ci_base[l] = h_lo[l];
            g->edges[l] = (h_hi[l] - h_lo[l]) / 2;
            nextb = h_rb[l];
        } else {
            g->group_base[l] = nextb;
            g->ci_base[l] = 0;
        }
        uint32_t Gl = g->G[l];
        g->H[l] = (g->flags & GSI_GRAPH_TEST_FEW_HOME_GROUPS) ? (Gl + GSI_PCSR_GPN - 1) / GSI_PCSR_GPN : Gl;
    }
    for (uint32_t l = 0; l < nlab; l++)
        if (g->G[l] == 0) g->ci_base[l] = 0;
    // device copy of the label table (one upload)
    uint64_t *d_tab = s.get<uint64_t>(3 * (uint64_t)nlab + 1, "label table");
    const uint64_t *d_rb = d_tab, *d_seg = d_tab + nlab;
    const uint32_t *d_G = reinterpret_cast<const uint32_t *>(d_tab + 2 * (uint64_t)nlab), *d_H = d_G + nlab;
    if (nlab) {
        // staged in pinned memory when it fits, else the copy is waited for
        const bool pin = 24ull * nlab <= 56 * 1024;
        std::vector<uint64_t> own(pin ? 0 : 3 * (uint64_t)nlab);
        uint64_t *t = pin ? c->pinned + 1024 : own.data();
        memcpy(t, g->group_base.data(), 8ull * nlab);
        memcpy(t + nlab, g->ci_base.data(), 8ull * nlab);
        memcpy(t + 2 * (uint64_t)nlab, g->G.data(), 4ull * nlab);
        memcpy(reinterpret_cast<uint32_t *>(t + 2 * (uint64_t)nlab) + nlab, g->H.data(), 4ull * nlab);
        GSI_HIP(hipMemcpyAsync(d_tab, t, 24ull * nlab, hipMemcpyHostToDevice, c->stream));
        if (!pin) sync(c);
    }
    LabelTab lt{d_rb, d_G, d_H, d_seg};

    g->gl = persist<uint32_t>(c, R * GROUP_WORDS, "pcsr groups");
    g->bytes = 4ull * GSI_SIG_WORDS * n + 4ull * nd + 4ull * GROUP_WORDS * R;

    if (R) {
        // home groups, stable sort of keys by group
        uint64_t *key = s.get<uint64_t>(R, "group key"), *key2 = s.get<uint64_t>(R, "group key tmp");
        uint32_t *cnt = s.get<uint32_t>(R, "home counts");
        fill_u32(c, cnt, 0, R);
        launch(c, "k_home", 20.0 * R, k_home, blocks(R), BT, run_vid, run_lab, R, lt, key, cnt);
        if (key_sort(c, (uint32_t)R, key, key2, 32, 32 + bits_for(R - 1), s)) std::swap(key, key2);
        const uint64_t *sorted = key;

        uint64_t *gstart = s.get<uint64_t>(R + 1, "group key start");
        exclusive_scan(c, cnt, R, gstart, s);
        uint32_t *need = s.get<uint32_t>(R, "overflow need");
        uint32_t *empt = s.get<uint32_t>(R, "empty flag");
        launch(c, "k_overflow_flags", 12.0 * R, k_overflow_flags, blocks(R), BT, cnt, R, need, empt);
        uint64_t *nscan = s.get<uint64_t>(R + 1, "need scan");
        uint64_t *escan = s.get<uint64_t>(R + 1, "empty scan");
        exclusive_scan(c, need, R, nscan, s);
        exclusive_scan(c, empt, R, escan, s);
        uint32_t *elist = s.get<uint32_t>(3 * R, "empty list, chains");
        uint32_t *next = elist + R, *owner = next + R;
        fill_u32(c, elist, NONE32, 3 * R);
        launch(c, "k_empty_list", 16.0 * R, k_empty_list, blocks(R), BT, empt, escan, R, d_rb, d_G, nlab, elist);
        launch(c, "k_claim1", 32.0 * nlab, k_claim1, blocks(nlab), BT, nscan, escan, d_rb, d_G, nlab, err);
        uint32_t *cidx = s.get<uint32_t>(R, "chain index");
        fill_u32(c, maxchain, 1, 1);
        launch(c, "k_chains", 12.0 * R, k_chains, blocks(R), BT, need, nscan, elist, R, d_rb, d_G, nlab, next, owner, cidx, maxchain);
        uint64_t *kfirst = s.get<uint64_t>(R, "group first key");
        uint32_t *nkeys = s.get<uint32_t>(R, "group keys");
        uint32_t *gdeg = s.get<uint32_t>(R, "group degree");
        launch(c, "k_group_keys", 32.0 * R, k_group_keys, blocks(R), BT, cnt, gstart, owner, cidx, sorted, run_start, R, nd, d_rb, d_G, nlab, kfirst, nkeys, gdeg);
        uint64_t *gci = s.get<uint64_t>(R + 1, "group ci start");
        exclusive_scan(c, gdeg, R, gci, s);
        uint32_t *run_off = keep_cr ? persist<uint32_t>(c, R, "cr offsets") : s.get<uint32_t>(R, "run offset");
        if (keep_cr) g->cr_off = run_off;
        launch(c, "k_write_groups", 128.0 * R + 24.0 * R, k_write_groups, blocks(R), BT, kfirst, nkeys, gci, next, sorted, run_start, run_vid, R, nd, d_rb, d_G, d_seg, nlab, g->gl, run_off);
        launch(c, "k_scatter_ci", 12.0 * nd, k_scatter_ci, nrt, BT, E, nd, (const uint64_t *)roff,
               (const uint32_t *)run_start, (const uint32_t *)run_off, d_seg, g->ci);
    }
    read_scalars(c, scal, hs, 3);
    if ((uint32_t)hs[0] & ERR_CLAIM1) fail(GSI_E_INTERNAL, "PCSR: not enough empty groups (Claim 1)");
    g->max_chain = R ? (uint32_t)hs[2] : 0;
    auto t1 = std::chrono::steady_clock::now();
    g->build_ms = std::chrono::duration<double, std::milli>(t1 - t0).count();
}

}  // namespace gsi
