// Level-synchronous joins of many queries at once.
//
// Every step advances each active query by one join level (Algorithm 3 with
// Algorithm 4's pre-allocation), all queries sharing the same launches:
//   rows      the tables of all active queries are one row space: query q
//             owns global rows [rbase_q, rbase_q + R_q)
//   k_wlocate one thread per global row: N(v, l) for every linking edge of
//             the row's own query; bound = |N(v', l0)|
//   scan      F over all rows -> one global slot space [0, |GBA|)
//   k_wjoin   groups of 256-slot tiles over the global slots: the same tests
//             as the single-query join, with each slot's query found from
//             its row; survivors as (element, row) records per group
//   scan      survivor offsets; k_wsurv turns them into each query's first
//             and last survivor, so every query's next table gets its exact
//             size (host readback)
//   k_wlink   a thread per survivor: (m_i, x) into the query's own next
//             table, or, at a query's last level, its rows in query-vertex
//             order, the rows' hashes summed per query
// When 8 bytes per slot do not fit the arena comfortably the join writes a
// keep bit per slot instead, and k_wlink_bits works on slot groups.
// Slots of a query are contiguous and ordered by its rows, so each query's
// result, row order included, equals the single-query path's.
#include <algorithm>
#include <chrono>
#include <cstring>

#include "join_device.h"
#include "scan_device.h"
#include "wide.h"

namespace gsi {

constexpr uint32_t WT = 256;

struct WEdge {
    const uint32_t *gl;
    const uint32_t *ci;
    uint32_t G, H, col;
    uint32_t ci_off;  // offset of its label's lists in the whole ci array
};

// Lookups of a query's rows at loc + locbase (even): (start, length) of
// linking edge e at words 2(e*R + i) and the next (one 8-byte load), start (in
// the array of scanned lists) of the list the row scans at [2ne*R + i] and
// that list's edge at [(2ne+1)*R + i].
struct WQ {
    const uint32_t *M;  // table, column c at M + c*R
    uint64_t R, rbase, locbase;
    const uint64_t *Cu;
    uint32_t j, ne, e0, efirst, k, final_level;
    uint32_t *Mn;   // next table (inner level)
    uint32_t *out;  // result rows (last level)
    uint64_t S, sbase;
    uint32_t qcol[GSI_MAX_K];
    uint32_t mmask;  // columns of m_i whose query vertex has u's label
    uint32_t pre;    // 1: the rows scan lists already filtered by C(u)
    const uint32_t *ci;  // array of the scanned lists: every label's, or the filtered ones
};

__device__ __forceinline__ uint2 wloc_pair(const WQ &Q, const uint32_t *loc, uint32_t e, uint64_t i) {
    return reinterpret_cast<const uint2 *>(loc + Q.locbase)[(uint64_t)e * Q.R + i];
}

// Candidates a join thread tests at once (wkeep_many), and the parts a
// search round splits a range in: as in the single-query join, two
// candidates fit the registers of 8 waves per SIMD, and 4-ary rounds with a
// vector tail issue fewer loads.
constexpr uint32_t WU = 2;
constexpr uint32_t WARITY = 4;

// x[u] not among N of the row's values, columns taken from the low bits of mm
template <uint32_t U, uint32_t N>
__device__ __forceinline__ void wdiffers(const WQ &Q, uint32_t &mm, const uint32_t *x, const uint64_t *i, bool *keep) {
    uint32_t cq[N], m[U][N];
#pragma unroll
    for (uint32_t t = 0; t < N; t++) {
        // past the last column it is read again
        cq[t] = (uint32_t)__builtin_ctz(mm);
        if (mm & (mm - 1)) mm &= mm - 1;
        else if (t + 1 == N) mm = 0;
    }
#pragma unroll
    for (uint32_t u = 0; u < U; u++)
#pragma unroll
        for (uint32_t t = 0; t < N; t++) m[u][t] = Q.M[(uint64_t)cq[t] * Q.R + i[u]];
#pragma unroll
    for (uint32_t u = 0; u < U; u++)
#pragma unroll
        for (uint32_t t = 0; t < N; t++) keep[u] = keep[u] && m[u][t] != x[u];
}

// The costly tests of U candidates of query Q at once (rows i[u] of Q's
// table): keep[u] (on entry: candidate u is live) becomes x[u] not in the
// row's values and x[u] in every other linking list of the row.  Every step
// issues the loads of all U candidates before using any.
template <uint32_t U>
__device__ __forceinline__ void wkeep_many(const WQ &Q, const uint32_t *loc, const WEdge *edges, const uint32_t *x,
                                           const uint64_t *i, bool *keep) {
    // only the columns of u's label can hold x; in chunks of 1, 2 or 4
    uint32_t mm = Q.mmask;
    while (mm) {
        const int left = __popc(mm);
        if (left >= 3) wdiffers<U, 4>(Q, mm, x, i, keep);
        else if (left == 2) wdiffers<U, 2>(Q, mm, x, i, keep);
        else wdiffers<U, 1>(Q, mm, x, i, keep);
    }
    if (Q.ne < 2) return;
    uint32_t be[U];
#pragma unroll
    for (uint32_t u = 0; u < U; u++) be[u] = loc[Q.locbase + (uint64_t)(2 * Q.ne + 1) * Q.R + i[u]];
    for (uint32_t e2 = 0; e2 < Q.ne; e2++) {
        uint32_t st[U], len[U];
        bool act[U], hit[U], any = false;
#pragma unroll
        for (uint32_t u = 0; u < U; u++) {
            act[u] = keep[u] && e2 != be[u];
            any |= act[u];
        }
        if (!any) continue;
#pragma unroll
        for (uint32_t u = 0; u < U; u++) {
            const uint2 sl = wloc_pair(Q, loc, e2, i[u]);
            st[u] = sl.x;
            len[u] = act[u] ? sl.y : 0u;
        }
        in_sorted_many<U, true, WARITY>(edges[Q.efirst + e2].ci, st, len, x, hit);
#pragma unroll
        for (uint32_t u = 0; u < U; u++)
            if (act[u]) keep[u] = hit[u];
    }
}

// Copies n words from the device and waits for the stream: through the
// pinned staging area when they fit (a pageable copy is staged by the
// runtime, several microseconds more).
static void read_words(gsi_ctx *c, const uint64_t *dev, std::vector<uint64_t> &out, uint64_t n) {
    out.resize(n);
    const bool pin = 8 * n <= 56 * 1024;
    uint64_t *dst = pin ? c->pinned + 1024 : out.data();
    GSI_HIP(hipMemcpyAsync(dst, dev, 8 * n, hipMemcpyDeviceToHost, c->stream));
    sync(c);
    if (pin) memcpy(out.data(), dst, 8 * n);
}

static uint32_t wblocks(uint64_t n) {
    uint64_t b = (n + WT - 1) / WT;
    if (b == 0) b = 1;
    if (b > 0x7FFFFFFFull) fail(GSI_E_CAPACITY, "grid too large");
    return (uint32_t)b;
}

// largest q in [lo, hi] with qs[q].rbase <= r
__device__ __forceinline__ uint32_t query_of(const WQ *qs, uint32_t lo, uint32_t hi, uint64_t r) {
    while (lo < hi) {
        uint32_t mid = (lo + hi + 1) >> 1;
        if (qs[mid].rbase <= r) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Each row scans its shortest linking list (e0's on ties): the survivors,
// and their order, are those of the first edge of Algorithm 4.
__global__ __launch_bounds__(WT) void k_wlocate(const WQ *qs, uint32_t nq, const WEdge *edges, uint64_t Rtot,
                                               uint32_t *loc, uint32_t *bound, uint32_t *rowq) {
    __shared__ uint32_t s_q[2];
    const uint64_t r0 = (uint64_t)blockIdx.x * WT;
    if (threadIdx.x == 0) {
        const uint64_t rl = r0 + WT - 1 < Rtot ? r0 + WT - 1 : Rtot - 1;
        s_q[0] = query_of(qs, 0, nq - 1, r0);
        s_q[1] = query_of(qs, s_q[0], nq - 1, rl);
    }
    __syncthreads();
    const uint64_t r = r0 + threadIdx.x;
    if (r >= Rtot) return;
    const uint32_t qi = query_of(qs, s_q[0], s_q[1], r);
    rowq[r] = qi;  // the row's query, for the join and link of this step
    const WQ &Q = qs[qi];
    const uint64_t i = r - Q.rbase;
    uint32_t s0 = 0, l0 = 0, ob = NONE32, os = 0, ol = 0xFFFFFFFFu;
    for (uint32_t e = 0; e < Q.ne; e++) {
        const WEdge &ed = edges[Q.efirst + e];
        const uint32_t v = Q.M[(uint64_t)ed.col * Q.R + i];
        const uint2 f = pcsr_find(ed.gl, ed.G, ed.H, v);
        reinterpret_cast<uint2 *>(loc + Q.locbase)[(uint64_t)e * Q.R + i] = f;
        if (e == Q.e0) {
            s0 = f.x;
            l0 = f.y;
        } else if (f.y < ol) {
            ob = e;
            os = f.x;
            ol = f.y;
        }
    }
    uint32_t be = Q.e0, bs = s0, bl = l0;
    if (ob != NONE32 && ol < l0) {
        be = ob;
        bs = os;
        bl = ol;
    }
    bound[r] = bl;
    loc[Q.locbase + (uint64_t)(2 * Q.ne) * Q.R + i] = edges[Q.efirst + be].ci_off + bs;
    loc[Q.locbase + (uint64_t)(2 * Q.ne + 1) * Q.R + i] = be;
}

// Level-wide filtered lists (the single-query path's, for the queries of a
// step whose rows scan far more list elements than their first edge's label
// holds): C(u) is tested once per element of the label's lists, the kept
// elements are compacted in order, all such queries' one after the other in
// one array, and the query's rows scan the compacted lists.  On the batch of
// 1,024 queries two thirds of the 3*10^9 slots are in 94 levels whose lists
// hold 1/8 as many elements.  Item t filters
// the lists of query q; its elements are padded to whole words, its words are
// [w0, w0 + words of el) and its workgroups start at b0 (elements) and rb0
// (rows).
struct WFilter {
    const uint32_t *ci;  // the label's lists
    uint64_t el, w0;
    uint32_t b0, rb0, q, pad;
};
constexpr uint32_t WF_TILES = 4;  // elements per thread
// directed entries of the first edge's label per |GBA| slot of the query
// above which its lists are filtered (the single-query path's factor)
constexpr double WF_FACTOR = 2.0;
// slots the filter has to save in a step: it costs about ten launches and a
// wait, 100 us, in which the join takes 2^24 slots (a batch of 48 queries
// with levels of up to 2^20 slots was 6 % slower with it)
constexpr uint64_t WF_MIN_SLOTS = 1ull << 24;

__device__ __forceinline__ uint32_t filter_item(const WFilter *f, uint32_t n, uint32_t b, bool rows) {
    uint32_t lo = 0, hi = n - 1;
    while (lo < hi) {
        const uint32_t mid = (lo + hi + 1) >> 1;
        if ((rows ? f[mid].rb0 : f[mid].b0) <= b) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

__global__ __launch_bounds__(WT) void k_wfn_bits(const WQ *qs, const WFilter *f, uint32_t nf, uint64_t *bits,
                                                uint32_t *wcnt) {
    const WFilter &I = f[filter_item(f, nf, blockIdx.x, false)];
    const uint64_t *Cu = qs[I.q].Cu;
    const uint64_t base = (uint64_t)(blockIdx.x - I.b0) * (WF_TILES * WT) + threadIdx.x;
    uint32_t x[WF_TILES];
    uint64_t cw[WF_TILES];
#pragma unroll
    for (uint32_t r = 0; r < WF_TILES; r++) {
        const uint64_t p = base + r * WT;
        x[r] = I.ci[p < I.el ? p : I.el - 1];
    }
#pragma unroll
    for (uint32_t r = 0; r < WF_TILES; r++) cw[r] = Cu[x[r] >> 6];
#pragma unroll
    for (uint32_t r = 0; r < WF_TILES; r++) {
        const uint64_t p = base + r * WT;
        const uint64_t m = __ballot(p < I.el && ((cw[r] >> (x[r] & 63)) & 1ull));
        if (lane_id() == 0 && p < I.el) {
            bits[I.w0 + (p >> 6)] = m;
            wcnt[I.w0 + (p >> 6)] = (uint32_t)__popcll(m);
        }
    }
}

__global__ __launch_bounds__(WT) void k_wfn_compact(const WFilter *f, uint32_t nf, const uint64_t *bits,
                                                   const uint64_t *wpre, uint32_t *fn) {
    const WFilter &I = f[filter_item(f, nf, blockIdx.x, false)];
    const uint64_t base = (uint64_t)(blockIdx.x - I.b0) * (WF_TILES * WT) + threadIdx.x;
#pragma unroll
    for (uint32_t r = 0; r < WF_TILES; r++) {
        const uint64_t p = base + r * WT;
        if (p >= I.el) continue;
        const uint64_t m = bits[I.w0 + (p >> 6)];
        if ((m >> (p & 63)) & 1ull) fn[wpre[I.w0 + (p >> 6)] + rank_below(m)] = I.ci[p];
    }
}

// every row of a filtered query scans its e0 list's members of C(u)
__global__ __launch_bounds__(WT) void k_wfn_relocate(const WQ *qs, const WFilter *f, uint32_t nf, const uint64_t *bits,
                                                    const uint64_t *wpre, uint32_t *loc, uint32_t *bound) {
    const WFilter &I = f[filter_item(f, nf, blockIdx.x, true)];
    const WQ &Q = qs[I.q];
    const uint64_t i = (uint64_t)(blockIdx.x - I.rb0) * WT + threadIdx.x;
    if (i >= Q.R) return;
    const uint2 sl = wloc_pair(Q, loc, Q.e0, i);
    const uint32_t st = sl.x, len = sl.y;
    // kept elements before position p of the item
    auto rank = [&](uint64_t p) -> uint64_t {
        const uint64_t w = I.w0 + (p >> 6);
        const uint32_t b = (uint32_t)(p & 63);
        return b ? wpre[w] + (uint64_t)__popcll(bits[w] & ((1ull << b) - 1)) : wpre[w];
    };
    const uint64_t fs = len ? rank(st) : 0, fe = len ? rank((uint64_t)st + len) : 0;
    bound[Q.rbase + i] = (uint32_t)(fe - fs);
    loc[Q.locbase + (uint64_t)(2 * Q.ne) * Q.R + i] = (uint32_t)fs;
    loc[Q.locbase + (uint64_t)(2 * Q.ne + 1) * Q.R + i] = Q.e0;
}

// |GBA| of each query: its rows' slots
__global__ __launch_bounds__(WT) void k_wgba(const WQ *qs, uint32_t nq, const uint64_t *F, uint64_t *out) {
    const uint32_t q = blockIdx.x * WT + threadIdx.x;
    if (q < nq) out[q] = F[qs[q].rbase + qs[q].R] - F[qs[q].rbase];
}

// The join of WJ_TILES consecutive 256-slot tiles (a group) per workgroup:
// each thread takes one slot of each tile and issues their loads together,
// and the set-up (rows staged in LDS) is paid once per group.  Outputs are
// the group's survivor records and count, or per 256-slot tile WT/64 bitmap
// words and a count.  When the rows fit (staged), each slot's row
// comes from a map built once per workgroup: each row after the first
// marks the slot where its slice starts (the largest row wins where empty
// rows share a start) and a max-scan carries the marks forward.
// (WJ_TILES by default; the batch schedule may pick 1, 2, 4 or 8, tuned)
// A group is a chain of about eight dependent loads, so what counts is how
// many groups a CU holds: a row's list start and first slot are kept as one
// 32-bit position (18.5 KB of LDS a group, 26.6 with both), the descriptor
// in scalar registers, two candidates a thread in 64 VGPRs: 8 waves per
// SIMD.  On the batch of 1,024 queries a step took 1.06 ms, with filtered
// lists 0.61, and with this 0.46.
constexpr uint32_t WJ_TILES = 4;

template <uint32_t TPW>
__global__ __launch_bounds__(WT) __attribute__((amdgpu_waves_per_eu(TPW <= 4 ? 8 : 4))) void k_wjoin(
    const WQ *__restrict__ qs, const uint32_t *__restrict__ rowq, const WEdge *__restrict__ edges,
    const uint64_t *__restrict__ F, const uint64_t *__restrict__ tile_row, uint64_t ntiles, uint64_t gba,
    const uint32_t *__restrict__ loc, uint64_t *bitmap, uint32_t *rec_x, uint32_t *rec_r, uint32_t *tile_cnt) {
    constexpr uint32_t TS = TPW * WT;
    __shared__ uint32_t s_row[TS];    // row (from r_lo) of each slot, staged groups
    __shared__ uint32_t s_base[TS];   // per row: position of the group's slot 0 in the scanned lists
    __shared__ uint32_t s_w[WT / 64];
    __shared__ uint32_t s_x[TS];      // elements that passed the C(u) test, compacted
    __shared__ uint32_t s_r[TS];      // and their rows (from r_lo)
    __shared__ uint16_t s_slot[TS];   // and their slots in the group
    __shared__ uint64_t s_keep[TS / 64];
    __shared__ uint32_t s_n;
    // tile_row and tile_cnt are kept per group with records, per tile without
    const uint64_t t0 = (uint64_t)blockIdx.x * (rec_x ? 1 : TPW);
    const uint64_t t1 = rec_x ? t0 + 1 : t0 + TPW < ntiles ? t0 + TPW : ntiles;
    const uint64_t p0 = (uint64_t)blockIdx.x * TS;
    const uint64_t r_lo = tile_row[t0], r_hi = tile_row[t1];
    const uint64_t nr = r_hi - r_lo + 1;
    const bool staged = nr <= TS;
    const uint32_t q0 = __builtin_amdgcn_readfirstlane(rowq[r_lo]), q1 = __builtin_amdgcn_readfirstlane(rowq[r_hi]);
    const bool one = q0 == q1;  // one query in the group: its descriptor is read with scalar loads
    const WQ &Q0 = qs[q0];
    if (threadIdx.x == 0) s_n = 0;
    if (threadIdx.x < TS / 64) s_keep[threadIdx.x] = 0;
#pragma unroll
    for (uint32_t k = 0; k < TPW; k++) s_row[threadIdx.x * TPW + k] = 0;
    __syncthreads();
    if (staged) {
        for (uint32_t r = threadIdx.x; r < nr; r += WT) {
            const uint64_t Fr = F[r_lo + r];
            uint32_t st;
            if (one) {
                st = loc[Q0.locbase + (uint64_t)(2 * Q0.ne) * Q0.R + (r_lo + r - Q0.rbase)];
            } else {
                const WQ &Q = qs[rowq[r_lo + r]];
                st = loc[Q.locbase + (uint64_t)(2 * Q.ne) * Q.R + (r_lo + r - Q.rbase)];
            }
            s_base[r] = st + (uint32_t)(p0 - Fr);
            // rows after the first start past p0 (the first holds slot p0)
            if (r > 0 && Fr - p0 < TS) atomicMax(&s_row[Fr - p0], r);
        }
        __syncthreads();
        block_max_scan<WT, TPW>(s_row, s_w);
    }
    const uint32_t lane = lane_id();
    // x = N(v'_i, l0)[p - F[i]] for the thread's slot of each tile (a slot past
    // |GBA| re-reads the last one), then the C(u) test; the slots that pass are
    // compacted so that the costly tests below run in dense waves
    const uint32_t last = gba - p0 < TS ? (uint32_t)(gba - p0) - 1 : TS - 1;
    uint32_t xs[TPW], rs[TPW];
    bool kp[TPW];
#pragma unroll
    for (uint32_t k = 0; k < TPW; k++) {
        const uint32_t own = k * WT + threadIdx.x;
        kp[k] = own <= last;
        const uint32_t sl = own <= last ? own : last;
        uint32_t pos;
        if (staged) {
            rs[k] = s_row[sl];
            pos = s_base[rs[k]] + sl;
        } else {
            const uint64_t p = p0 + sl;
            uint64_t lo = r_lo, hi = r_hi;
            while (lo < hi) {
                const uint64_t mid = lo + (hi - lo + 1) / 2;
                if (F[mid] <= p) lo = mid;
                else hi = mid - 1;
            }
            rs[k] = (uint32_t)(lo - r_lo);
            const WQ &Q = qs[rowq[lo]];
            pos = loc[Q.locbase + (uint64_t)(2 * Q.ne) * Q.R + (lo - Q.rbase)] + (uint32_t)(p - F[lo]);
        }
        xs[k] = one ? Q0.ci[pos] : qs[rowq[r_lo + rs[k]]].ci[pos];
    }
    if (!(one && Q0.pre)) {
        // every slot's C(u) word is loaded before any is tested (a filtered
        // list's elements pass)
        uint64_t cw[TPW];
#pragma unroll
        for (uint32_t k = 0; k < TPW; k++) cw[k] = (one ? Q0.Cu : qs[rowq[r_lo + rs[k]]].Cu)[xs[k] >> 6];
#pragma unroll
        for (uint32_t k = 0; k < TPW; k++) kp[k] = kp[k] && ((cw[k] >> (xs[k] & 63)) & 1ull);
    }
#pragma unroll
    for (uint32_t k = 0; k < TPW; k++) {
        const uint64_t pm = __ballot(kp[k]);
        if (pm) {
            uint32_t base = 0;
            if (lane == 0) base = atomicAdd(&s_n, (uint32_t)__popcll(pm));
            base = __shfl(base, 0, 64);
            if (kp[k]) {
                const uint32_t idx = base + rank_below(pm);
                s_slot[idx] = (uint16_t)(k * WT + threadIdx.x);
                s_x[idx] = xs[k];
                s_r[idx] = rs[k];
            }
        }
    }
    __syncthreads();
    const uint32_t n = __builtin_amdgcn_readfirstlane(s_n);
    if (one) {
        // WU candidates per thread at a time, their loads issued together
        for (uint32_t e0 = 0; e0 < n; e0 += WU * WT) {
            uint32_t xs2[WU], sl[WU];
            uint64_t is[WU];
            bool kq[WU];
#pragma unroll
            for (uint32_t u = 0; u < WU; u++) {
                const uint32_t e = e0 + u * WT + threadIdx.x;
                kq[u] = e < n;
                const uint32_t c = kq[u] ? e : 0u;  // a past-the-end thread reads candidate 0
                sl[u] = s_slot[c];
                xs2[u] = s_x[c];
                is[u] = r_lo + s_r[c] - Q0.rbase;
            }
            wkeep_many<WU>(Q0, loc, edges, xs2, is, kq);
#pragma unroll
            for (uint32_t u = 0; u < WU; u++)
                if (kq[u]) atomicOr(&s_keep[sl[u] >> 6], 1ull << (sl[u] & 63));
        }
    }
    for (uint32_t e = one ? n : threadIdx.x; e < n; e += WT) {
        const uint32_t slot = s_slot[e], xv = s_x[e];
        const uint64_t r = r_lo + s_r[e];
        const WQ &Q = qs[rowq[r]];
        const uint64_t i = r - Q.rbase;
        bool keep = true;
        // x not in m_i: the row's values eight at a time, every load issued
        // before the compares (a column past j re-reads column j - 1)
        for (uint32_t c = 0; keep && c < Q.j; c += 8) {
            uint32_t m[8];
#pragma unroll
            for (uint32_t q = 0; q < 8; q++) m[q] = Q.M[(uint64_t)(c + q < Q.j ? c + q : Q.j - 1) * Q.R + i];
#pragma unroll
            for (uint32_t q = 0; q < 8; q++) keep = keep && m[q] != xv;
        }
        const uint32_t be = (keep && Q.ne > 1) ? loc[Q.locbase + (uint64_t)(2 * Q.ne + 1) * Q.R + i] : Q.e0;
        for (uint32_t e2 = 0; keep && e2 < Q.ne; e2++) {
            if (e2 == be) continue;
            const uint2 sl = wloc_pair(Q, loc, e2, i);
            keep = in_sorted(edges[Q.efirst + e2].ci + sl.x, sl.y, xv);
        }
        if (keep) atomicOr(&s_keep[slot >> 6], 1ull << (slot & 63));
    }
    __syncthreads();
    if (rec_x) {
        // the group's survivors as records in slot order (element, row from
        // r_lo): every kept slot is among the compacted candidates
        __shared__ uint32_t s_pre[(TPW * WT) / 64];
        if (threadIdx.x < 64) {
            const uint32_t c = threadIdx.x < (TPW * WT) / 64 ? (uint32_t)__popcll(s_keep[threadIdx.x]) : 0u;
            const uint32_t inc = wave_inclusive_sum(c);
            if (threadIdx.x < (TPW * WT) / 64) s_pre[threadIdx.x] = inc - c;
            if (threadIdx.x == 63) tile_cnt[blockIdx.x] = inc;
        }
        __syncthreads();
        for (uint32_t e = threadIdx.x; e < n; e += WT) {
            const uint32_t sl = s_slot[e];
            const uint64_t word = s_keep[sl >> 6];
            if ((word >> (sl & 63)) & 1ull) {
                const uint64_t q = p0 + s_pre[sl >> 6] + (uint32_t)__popcll(word & ((1ull << (sl & 63)) - 1));
                rec_x[q] = s_x[e];
                rec_r[q] = s_r[e];
            }
        }
        return;
    }
    // per 256-slot tile: its WT/64 bitmap words and their count
    if (threadIdx.x < 64) {
        const uint32_t tk = threadIdx.x / (WT / 64);  // tile of the group
        const uint64_t word = threadIdx.x < (TPW * WT) / 64 ? s_keep[threadIdx.x] : 0ull;
        if (threadIdx.x < (TPW * WT) / 64 && t0 + tk < t1) bitmap[p0 / 64 + threadIdx.x] = word;
        uint32_t c = (uint32_t)__popcll(word);
#pragma unroll
        for (uint32_t o = 1; o < WT / 64; o <<= 1) c += __shfl_xor(c, o, 64);
        if (threadIdx.x < (TPW * WT) / 64 && threadIdx.x % (WT / 64) == 0 && t0 + tk < t1) tile_cnt[t0 + tk] = c;
    }
}

// survivors before slot p
__device__ __forceinline__ uint64_t survivors_before(const uint64_t *bitmap, const uint64_t *tile_off, uint64_t gba,
                                                     uint64_t p) {
    const uint64_t ntiles = (gba + WT - 1) / WT;
    if (p >= gba) return tile_off[ntiles];
    const uint64_t t = p / WT;
    const uint32_t within = (uint32_t)(p - t * WT);
    uint64_t r = tile_off[t];
    for (uint32_t w = 0; w < within / 64; w++) r += (uint64_t)__popcll(bitmap[t * (WT / 64) + w]);
    const uint32_t b = within % 64;
    if (b) r += (uint64_t)__popcll(bitmap[t * (WT / 64) + within / 64] & ((1ull << b) - 1));
    return r;
}

// survivors of rows before r, p being the first slot of row r: those of the
// groups before p's and the records of p's group with an earlier row (rows
// ascend within a group)
__device__ __forceinline__ uint64_t records_before(const uint32_t *rec_r, const uint64_t *tile_row,
                                                   const uint64_t *tile_off, uint64_t ngroups, uint32_t group,
                                                   uint64_t p, uint64_t r) {
    const uint64_t g = p / group;
    if (g >= ngroups) return tile_off[ngroups];
    uint32_t lo = 0, hi = (uint32_t)(tile_off[g + 1] - tile_off[g]);
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (tile_row[g] + rec_r[g * group + mid] < r) lo = mid + 1;
        else hi = mid;
    }
    return tile_off[g] + lo;
}

// per query: first survivor, end of its survivors, first slot, end of slots
__global__ __launch_bounds__(WT) void k_wsurv(const WQ *qs, uint32_t nq, const uint64_t *F, const uint64_t *bitmap,
                                             const uint32_t *rec_r, const uint64_t *tile_row, uint64_t ntiles,
                                             uint32_t group, const uint64_t *tile_off, uint64_t gba, uint64_t *sb) {
    const uint32_t q = blockIdx.x * WT + threadIdx.x;
    if (q >= nq) return;
    const WQ &Q = qs[q];
    const uint64_t f0 = F[Q.rbase], f1 = F[Q.rbase + Q.R];
    if (rec_r) {
        sb[4 * (uint64_t)q] = records_before(rec_r, tile_row, tile_off, ntiles, group, f0, Q.rbase);
        sb[4 * (uint64_t)q + 1] = records_before(rec_r, tile_row, tile_off, ntiles, group, f1, Q.rbase + Q.R);
    } else {
        sb[4 * (uint64_t)q] = survivors_before(bitmap, tile_off, gba, f0);
        sb[4 * (uint64_t)q + 1] = survivors_before(bitmap, tile_off, gba, f1);
    }
    sb[4 * (uint64_t)q + 2] = f0;
    sb[4 * (uint64_t)q + 3] = f1;
}

// last-level rows of a one-query tile are staged in LDS and written as one
// contiguous block when k is at most this
constexpr uint32_t WLINK_STAGE_K = 16;

// Digests: every query has WACC (sum, xor) accumulators, the workgroups
// adding to them in turn, so that a query with many survivors does not have
// all of them at one address.
constexpr uint32_t WACC = 16;
__device__ __forceinline__ void add_hash(unsigned long long *acc, uint32_t q, uint64_t sum, uint64_t xr) {
    unsigned long long *a = acc + 2 * ((uint64_t)q * WACC + blockIdx.x % WACC);
    atomicAdd(a, (unsigned long long)sum);
    atomicXor(a + 1, (unsigned long long)xr);
}
__device__ __forceinline__ void add_hash(unsigned long long *acc, uint32_t q, uint64_t h) { add_hash(acc, q, h, h); }

// one thread per query: its accumulators into dig[2q], dig[2q + 1]
__global__ __launch_bounds__(WT) void k_wdigest(const uint64_t *acc, uint32_t nq, uint64_t *dig) {
    const uint32_t q = blockIdx.x * WT + threadIdx.x;
    if (q >= nq) return;
    uint64_t sm = 0, xr = 0;
#pragma unroll
    for (uint32_t t = 0; t < WACC; t++) {
        sm += acc[2 * ((uint64_t)q * WACC + t)];
        xr ^= acc[2 * ((uint64_t)q * WACC + t) + 1];
    }
    dig[2 * (uint64_t)q] = sm;
    dig[2 * (uint64_t)q + 1] = xr;
}

// The survivor's row of query Q (its row i of M, extended by x) into its
// place: the next table, or at the last level the staged or direct result
// row and, returned, its hash.  Values are loaded eight at a time, every load
// issued before any is used (a column past the end re-reads a valid one).
__device__ __forceinline__ uint64_t link_row(const WQ &Q, uint64_t i, uint32_t x, uint64_t pos, uint32_t *staged) {
    if (!Q.final_level) {
        for (uint32_t c = 0; c < Q.j; c += 8) {
            uint32_t m[8];
#pragma unroll
            for (uint32_t t = 0; t < 8; t++) m[t] = Q.M[(uint64_t)(c + t < Q.j ? c + t : Q.j - 1) * Q.R + i];
#pragma unroll
            for (uint32_t t = 0; t < 8; t++)
                if (c + t < Q.j) Q.Mn[(uint64_t)(c + t) * Q.S + pos] = m[t];
        }
        Q.Mn[(uint64_t)Q.j * Q.S + pos] = x;
        return 0;
    }
    uint64_t f = 14695981039346656037ull;
    for (uint32_t u0 = 0; u0 < Q.k; u0 += 8) {
        uint32_t val[8];
#pragma unroll
        for (uint32_t t = 0; t < 8; t++) {
            const uint32_t c = u0 + t < Q.k ? Q.qcol[u0 + t < GSI_MAX_K ? u0 + t : GSI_MAX_K - 1] : Q.j;
            const uint32_t mv = Q.M[(uint64_t)(c < Q.j ? c : 0u) * Q.R + i];
            val[t] = c < Q.j ? mv : x;
        }
#pragma unroll
        for (uint32_t t = 0; t < 8; t++) {
            const uint32_t u = u0 + t;
            if (u >= Q.k) break;
            if (staged) staged[u] = val[t];
            else if (Q.out) Q.out[pos * Q.k + u] = val[t];
            f = fnv_word(f, val[t]);
        }
    }
    return mix64(f);
}

// The link over survivor records, a thread per survivor (grid over the
// step's survivors, not its slots: one slot in 15 survives on a batch of
// 1,024 queries over 10^6 vertices, and workgroups over 1,024 slots had a
// quarter of their threads busy; there 1.24 -> 0.30 ms a step, digests
// included 1.33 -> 0.30).  stile[b] is the group that holds survivor WT * b.  A workgroup
// whose survivors are one query's reads that query's descriptor with scalar
// loads, stages its last-level rows in LDS (ROWS) and adds one digest.
template <bool ROWS>
__global__ __launch_bounds__(WT) void k_wlink(const WQ *__restrict__ qs, const uint32_t *rowq,
                                             const uint64_t *tile_row, const uint64_t *tile_off,
                                             const uint64_t *stile, uint32_t group, const uint32_t *rec_x,
                                             const uint32_t *rec_r, uint64_t S, unsigned long long *acc) {
    __shared__ uint32_t s_q[2];
    __shared__ uint64_t s_d[2][WT / 64];
    __shared__ uint32_t s_rows[ROWS ? WT * WLINK_STAGE_K : 1];
    const uint64_t s0 = (uint64_t)blockIdx.x * WT;
    const uint32_t n = S - s0 < WT ? (uint32_t)(S - s0) : WT;  // survivors of the workgroup
    const bool mine = threadIdx.x < n;
    const uint64_t gpos = s0 + (mine ? threadIdx.x : 0u);
    uint64_t g = stile[blockIdx.x];
    uint64_t hi = stile[blockIdx.x + 1];
    while (g < hi) {
        const uint64_t mid = g + (hi - g + 1) / 2;
        if (tile_off[mid] <= gpos) g = mid;
        else hi = mid - 1;
    }
    const uint64_t at = g * group + (gpos - tile_off[g]);
    const uint32_t x = rec_x[at];
    const uint64_t r = tile_row[g] + rec_r[at];
    const uint32_t qi = rowq[r];
    if (threadIdx.x == 0) s_q[0] = qi;
    if (threadIdx.x == n - 1) s_q[1] = qi;
    __syncthreads();
    const uint32_t q0 = __builtin_amdgcn_readfirstlane(s_q[0]), q1 = __builtin_amdgcn_readfirstlane(s_q[1]);
    if (q0 != q1) {
        // survivors of several queries
        if (mine) {
            const WQ &Q = qs[qi];
            const uint64_t pos = gpos - Q.sbase;
            if (pos < Q.S) {  // always, when the survivor ranges are consistent
                const uint64_t h = link_row(Q, r - Q.rbase, x, pos, nullptr);
                if (Q.final_level) add_hash(acc, qi, h);
            }
        }
        return;
    }
    const WQ &Q = qs[q0];
    const bool stage = ROWS && Q.final_level && Q.k <= WLINK_STAGE_K;
    const uint64_t pos = gpos - Q.sbase;
    uint64_t h = 0;
    if (mine && pos < Q.S) h = link_row(Q, r - Q.rbase, x, pos, stage ? s_rows + threadIdx.x * Q.k : nullptr);
    if (!Q.final_level) return;
    const uint64_t sum = wave_sum(h), xr = wave_xor(h);
    if (lane_id() == 0) {
        s_d[0][threadIdx.x >> 6] = sum;
        s_d[1][threadIdx.x >> 6] = xr;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t ts = 0, tx = 0;
#pragma unroll
        for (uint32_t t = 0; t < WT / 64; t++) {
            ts += s_d[0][t];
            tx ^= s_d[1][t];
        }
        add_hash(acc, q0, ts, tx);
    }
    if (stage) {
        // the workgroup's rows are one contiguous block of the result
        const uint64_t first = s0 - Q.sbase;
        uint64_t end = first + n;
        if (end > Q.S) end = Q.S;
        const uint32_t nw = first < end ? (uint32_t)(end - first) * Q.k : 0u;
        uint32_t *dst = Q.out + first * Q.k;
        for (uint32_t v = threadIdx.x; v < nw; v += WT) dst[v] = s_rows[v];
    }
}

// The same from keep bits, for steps whose records would not fit.  A workgroup
// takes the same WJ_TILES consecutive tiles as the join: their kept slots
// are listed in slot order in LDS first, so that the waves that gather,
// write and hash are dense, and survivor q of the list is survivor
// tile_off[t0] + q of the step.  The row of a survivor's slot is found by a
// binary search over the group's rows in LDS (survivors are often few, so
// a map of every slot would not pay).
template <uint32_t TPW>
__global__ __launch_bounds__(WT) void k_wlink_bits(const WQ *qs, const uint32_t *rowq,
                                             const uint64_t *F, const uint64_t *tile_row, uint64_t ntiles,
                                             const uint32_t *loc, const uint64_t *bitmap, const uint64_t *tile_off,
                                             unsigned long long *acc) {
    __shared__ uint64_t s_F[(TPW * WT)];
    __shared__ uint32_t s_st[(TPW * WT)];
    __shared__ WQ s_Q;
    __shared__ uint32_t s_q[2];
    __shared__ uint32_t s_rows[WT * WLINK_STAGE_K];
    __shared__ uint16_t s_list[(TPW * WT)];          // the group's kept slots, in slot order
    __shared__ uint32_t s_pre[(TPW * WT) / 64 + 1];  // kept slots before each bitmap word
    const uint64_t t0 = (uint64_t)blockIdx.x * TPW;
    const uint64_t t1 = t0 + TPW < ntiles ? t0 + TPW : ntiles;
    const uint64_t gbase = tile_off[t0];
    if (tile_off[t1] == gbase) return;  // no survivor in the group (uniform)
    const uint64_t p0 = t0 * WT;
    const uint32_t nwords = (uint32_t)(t1 - t0) * (WT / 64);
    const uint64_t *words = bitmap + p0 / 64;
    const uint64_t r_lo = tile_row[t0], r_hi = tile_row[t1];
    const uint64_t nr = r_hi - r_lo + 1;
    const bool staged = nr <= (TPW * WT);
    if (threadIdx.x == 0) {
        s_q[0] = rowq[r_lo];
        s_q[1] = rowq[r_hi];
        uint32_t run = 0;
        for (uint32_t q = 0; q < (TPW * WT) / 64; q++) {
            s_pre[q] = run;
            if (q < nwords) run += (uint32_t)__popcll(words[q]);
        }
        s_pre[(TPW * WT) / 64] = run;
    }
    if (staged)
        for (uint32_t r = threadIdx.x; r < nr; r += WT) s_F[r] = F[r_lo + r];
    __syncthreads();
    const bool one = s_q[0] == s_q[1];
    if (one) {
        const WQ &Q = qs[s_q[0]];
        const uint32_t *src = reinterpret_cast<const uint32_t *>(&Q);
        uint32_t *dst = reinterpret_cast<uint32_t *>(&s_Q);
        for (uint32_t w = threadIdx.x; w < sizeof(WQ) / 4; w += WT) dst[w] = src[w];
        if (staged)
            for (uint32_t r = threadIdx.x; r < nr; r += WT)
                s_st[r] = loc[Q.locbase + (uint64_t)(2 * Q.ne) * Q.R + (r_lo + r - Q.rbase)];
    }
    {
        const uint32_t w = threadIdx.x >> 6, lane = lane_id();
#pragma unroll
        for (uint32_t k = 0; k < TPW; k++) {
            const uint32_t wi = k * (WT / 64) + w;
            const uint64_t word = wi < nwords ? words[wi] : 0ull;
            if ((word >> lane) & 1ull) s_list[s_pre[wi] + rank_below(word)] = (uint16_t)(k * WT + threadIdx.x);
        }
    }
    __syncthreads();
    // the same count in every lane (the loop holds barriers)
    const uint32_t n = __builtin_amdgcn_readfirstlane(s_pre[(TPW * WT) / 64]);
    const bool stage = one && s_Q.final_level && s_Q.out && s_Q.k <= WLINK_STAGE_K;
    uint64_t hs = 0, hx = 0;
    for (uint32_t q0 = 0; q0 < n; q0 += WT) {
        const uint32_t local = threadIdx.x;  // survivor q0 + local of the group
        const uint32_t q = q0 + local;
        const uint64_t gpos = gbase + q;
        if (q < n) {
            const uint64_t p = p0 + s_list[q];
            uint64_t r, Fr;
            uint32_t lr = 0;
            if (staged) {
                uint32_t lo = 0, hi = (uint32_t)(nr - 1);
                while (lo < hi) {
                    const uint32_t mid = (lo + hi + 1) >> 1;
                    if (s_F[mid] <= p) lo = mid;
                    else hi = mid - 1;
                }
                lr = lo;
                r = r_lo + lo;
                Fr = s_F[lo];
            } else {
                uint64_t lo = r_lo, hi = r_hi;
                while (lo < hi) {
                    const uint64_t mid = lo + (hi - lo + 1) / 2;
                    if (F[mid] <= p) lo = mid;
                    else hi = mid - 1;
                }
                r = lo;
                Fr = F[lo];
            }
            const WQ &Q = one ? s_Q : qs[rowq[r]];
            const uint64_t i = r - Q.rbase;
            const uint64_t pos = gpos - Q.sbase;
            if (pos < Q.S) {  // always, when the survivor ranges are consistent
                const uint32_t st0 = (one && staged) ? s_st[lr] : loc[Q.locbase + (uint64_t)(2 * Q.ne) * Q.R + i];
                const uint32_t x = Q.ci[st0 + (uint32_t)(p - Fr)];
                const uint64_t h = link_row(Q, i, x, pos, stage ? s_rows + local * Q.k : nullptr);
                if (Q.final_level) {
                    if (one) {
                        hs += h;
                        hx ^= h;
                    } else {
                        add_hash(acc, rowq[r], h);
                    }
                }
            }
        }
        if (stage) {
            // the round's rows are one contiguous block of the query's result
            __syncthreads();
            const uint64_t first = gbase + q0 - s_Q.sbase;
            uint64_t end = gbase + (q0 + WT < n ? q0 + WT : n) - s_Q.sbase;
            if (end > s_Q.S) end = s_Q.S;
            const uint32_t nw = first < end ? (uint32_t)(end - first) * s_Q.k : 0u;
            uint32_t *dst = s_Q.out + first * s_Q.k;
            for (uint32_t v = threadIdx.x; v < nw; v += WT) dst[v] = s_rows[v];
            __syncthreads();
        }
    }
    if (one && s_Q.final_level) {
        hs = wave_sum(hs);
        hx = wave_xor(hx);
        if (lane_id() == 0) add_hash(acc, s_q[0], hs, hx);
    }
}

// One join level for the queries in `act` (all of them, or none: on an
// allocation failure everything allocated for the step is given back and
// no query changes state).  records: survivors as records where they fit;
// filter: lists rescanned many times over are filtered first.
static void wide_step(gsi_graph *g, const std::vector<WideQuery *> &act, bool count_only, uint32_t tpw, bool records,
                      bool filter) {
    gsi_ctx *c = g->ctx;
    {
        const uint32_t nq = (uint32_t)act.size();
        Scratch s(c);
        std::vector<WQ> hq(nq);
        std::vector<WEdge> he;
        std::vector<WFilter> fl;  // lists filtered this step
        // per-step allocations of the queries, released unless the step
        // commits; declared after the host arrays so that, on a failure, the
        // stream has drained the copies out of them before they go
        struct Pending {
            std::vector<WideQuery *> q;
            bool commit = false;
            gsi_ctx *c;
            ~Pending() {
                if (commit) return;
                (void)hipStreamSynchronize(c->stream);
                for (auto *x : q) {
                    if (x->next) c->arena.release(x->next);
                    x->next = nullptr;
                    if (x->rows) c->arena.release(x->rows);
                    x->rows = nullptr;
                    x->digest[0] = x->digest[1] = 0;
                }
            }
        } pend;
        pend.q = act;
        pend.c = c;
        uint64_t Rtot = 0, loctot = 0;
        std::vector<uint32_t> lab0(nq, 0);  // label of the first edge
        double least = 1e300;               // |GBA| from which any query's lists would be filtered
        for (uint32_t a = 0; a < nq; a++) {
            WideQuery &x = *act[a];
            const HostQuery &q = *x.q;
            const uint32_t j = x.j, u = x.order[j];
            WQ &Q = hq[a];
            memset(&Q, 0, sizeof(Q));
            Q.M = x.M;
            Q.R = x.R;
            Q.rbase = Rtot;
            Q.Cu = x.Cu[j];
            Q.j = j;
            Q.k = q.k;
            Q.final_level = j == q.k - 1;
            Q.efirst = (uint32_t)he.size();
            for (uint32_t i = 0; i < j; i++)
                for (auto &p : q.adj[u])
                    if (p.first == x.order[i]) {
                        const uint32_t l = p.second;
                        WEdge ed;
                        ed.gl = g->gl + g->group_base[l] * GROUP_WORDS;
                        ed.ci = g->ci + g->ci_base[l];
                        ed.G = g->G[l];
                        ed.H = g->H[l];
                        ed.col = i;
                        ed.ci_off = (uint32_t)g->ci_base[l];
                        if (x.order[i] == x.e0src[j]) {
                            Q.e0 = Q.ne;
                            lab0[a] = l;
                        }
                        he.push_back(ed);
                        Q.ne++;
                    }
            Q.ci = g->ci;
            least = std::min(least, WF_FACTOR * 2.0 * (double)g->edges[lab0[a]]);
            Q.locbase = loctot;
            for (uint32_t v = 0; v < q.k; v++) Q.qcol[v] = x.col[v];
            for (uint32_t c = 0; c < j; c++)
                if (q.multi || q.vl[x.order[c]] == q.vl[u]) Q.mmask |= 1u << c;
            x.stats_rows[j] = x.R;
            Rtot += x.R;
            loctot += (2ull * Q.ne + 2) * x.R;
        }
        WQ *d_q = s.get<WQ>(nq, "wide queries");
        WEdge *d_e = s.get<WEdge>(he.size(), "wide edges");
        uint32_t *loc = s.get<uint32_t>(loctot, "wide lookups");
        uint32_t *bound = s.get<uint32_t>(Rtot, "wide bounds");
        uint32_t *rowq = s.get<uint32_t>(Rtot, "wide row queries");
        uint64_t *F = s.get<uint64_t>(Rtot + 1, "wide offsets F");
        uint64_t *scal = c->mbox_dev + MBOX_SCALARS;  // read by the host without a copy
        GSI_HIP(hipMemcpyAsync(d_q, hq.data(), sizeof(WQ) * nq, hipMemcpyHostToDevice, c->stream));
        GSI_HIP(hipMemcpyAsync(d_e, he.data(), sizeof(WEdge) * he.size(), hipMemcpyHostToDevice, c->stream));
        double lb = 0;
        for (auto &Q : hq) lb += (double)Q.R * (4.0 * Q.ne + 128.0 * Q.ne + 8.0 * Q.ne + 4.0);
        launch(c, "k_wlocate", lb, k_wlocate, wblocks(Rtot), WT, (const WQ *)d_q, nq, (const WEdge *)d_e, Rtot, loc,
               bound, rowq);
        exclusive_scan(c, bound, Rtot, F, s, scal);
        uint64_t gba;
        read_scalars(c, scal, &gba, 1);  // also orders the uploads above before `hq`/`he` change
        if (gba == 0) {
            pend.commit = true;
            for (auto *x : act) {
                x->stats_gba[x->j] = 0;
                x->levels = x->j;
                x->finish_empty();
            }
            return;
        }
        // queries whose rows rescan their first edge's lists many times over:
        // filter those lists by C(u) once
        if (filter && (double)gba > least && gba >= WF_MIN_SLOTS) {
            std::vector<uint64_t> qg;
            uint64_t *d_qg = s.get<uint64_t>(nq, "wide slots per query");
            launch(c, "k_wgba", 16.0 * nq, k_wgba, wblocks(nq), WT, (const WQ *)d_q, nq, (const uint64_t *)F, d_qg);
            read_words(c, d_qg, qg, nq);
            uint64_t words = 0, els = 0, blk = 0, rblk = 0, saved = 0;
            const uint64_t room = c->arena.largest_free() / 4;
            for (uint32_t a = 0; a < nq; a++) {
                const uint32_t l = lab0[a];
                const uint64_t el = 2 * g->edges[l];
                if (el == 0 || (double)qg[a] <= WF_FACTOR * (double)el) continue;
                // positions in the compacted array are 32-bit
                if (els + el >= 0xFFFFFFFFull || 5 * (els + el) + 4096 > room) continue;
                WFilter f{g->ci + g->ci_base[l], el, words, (uint32_t)blk, (uint32_t)rblk, a, 0};
                words += (el + 63) / 64 + 1;  // one spare word: a list may end at the label's last element
                els += el;
                saved += qg[a] - el;
                blk += (el + WF_TILES * WT - 1) / (WF_TILES * WT);
                rblk += (hq[a].R + WT - 1) / WT;
                fl.push_back(f);
            }
            if (saved >= WF_MIN_SLOTS) {
                const uint32_t nf = (uint32_t)fl.size();
                WFilter *d_f = s.get<WFilter>(nf, "wide filters");
                uint64_t *fbits = s.get<uint64_t>(words, "filtered-list bits");
                uint32_t *wcnt = s.get<uint32_t>(words, "filtered-list word counts");
                uint64_t *wpre = s.get<uint64_t>(words + 1, "filtered-list word offsets");
                uint32_t *fn = s.get<uint32_t>(els, "filtered lists");
                GSI_HIP(hipMemcpyAsync(d_f, fl.data(), sizeof(WFilter) * nf, hipMemcpyHostToDevice, c->stream));
                fill_u32(c, wcnt, 0, words);  // the spare words
                launch(c, "k_fn_bits", 4.0 * els, k_wfn_bits, (uint32_t)blk, WT, (const WQ *)d_q, (const WFilter *)d_f,
                       nf, fbits, wcnt);
                exclusive_scan(c, wcnt, words, wpre, s);
                launch(c, "k_fn_compact", 4.0 * els, k_wfn_compact, (uint32_t)blk, WT, (const WFilter *)d_f, nf,
                       (const uint64_t *)fbits, (const uint64_t *)wpre, fn);
                launch(c, "k_fn_relocate", 52.0 * WT * rblk, k_wfn_relocate, (uint32_t)rblk, WT, (const WQ *)d_q,
                       (const WFilter *)d_f, nf, (const uint64_t *)fbits, (const uint64_t *)wpre, loc, bound);
                exclusive_scan(c, bound, Rtot, F, s, scal);
                for (auto &f : fl) {
                    hq[f.q].pre = 1;
                    hq[f.q].ci = fn;
                }
                GSI_HIP(hipMemcpyAsync(d_q, hq.data(), sizeof(WQ) * nq, hipMemcpyHostToDevice, c->stream));
                read_scalars(c, scal, &gba, 1);  // also orders the uploads above
                if (gba == 0) {
                    pend.commit = true;
                    for (auto *x : act) {
                        x->levels = x->j;
                        x->finish_empty();
                    }
                    return;
                }
            }
        }
        // survivor records per group of tpw tiles when they fit comfortably
        // (8 bytes per slot), else keep bits per tile
        const uint32_t group = tpw * WT;
        const uint64_t ngroups = (gba + group - 1) / group;
        const bool recs = records && 8.0 * (double)(ngroups * group) <= (double)c->arena.largest_free() / 4;
        const uint64_t ntiles = recs ? ngroups : (gba + WT - 1) / WT;
        uint32_t *rec_x = nullptr, *rec_r = nullptr;
        uint64_t *bitmap = nullptr;
        if (recs) {
            rec_x = s.get<uint32_t>(ngroups * group, "wide survivor elements");
            rec_r = s.get<uint32_t>(ngroups * group, "wide survivor rows");
        } else {
            bitmap = s.get<uint64_t>(ntiles * (WT / 64), "wide GBA bitmap");
        }
        uint64_t *trow = s.get<uint64_t>(ntiles + 1, "wide tile rows");
        uint32_t *tcnt = s.get<uint32_t>(ntiles, "wide tile counts");
        uint64_t *toff = s.get<uint64_t>(ntiles + 1, "wide tile offsets");
        uint64_t *sb = s.get<uint64_t>(4ull * nq, "wide survivor ranges");
        tile_rows(c, F, Rtot, ntiles, recs ? group : WT, trow);
        double jb = 4.0 * gba + (recs ? 0.0 : gba / 8.0) + 4.0 * ntiles;
        for (auto &Q : hq) jb += (double)Q.R * (8.0 + 8.0 * Q.ne + 4.0 * Q.j);
        {
            auto join = [&](auto kern) {
                launch(c, "k_wjoin", jb, kern, (uint32_t)ngroups, WT, (const WQ *)d_q, (const uint32_t *)rowq,
                       (const WEdge *)d_e, (const uint64_t *)F, (const uint64_t *)trow, ntiles,
                       gba, (const uint32_t *)loc, bitmap, rec_x, rec_r, tcnt);
            };
            if (tpw == 1) join(k_wjoin<1>);
            else if (tpw == 2) join(k_wjoin<2>);
            else if (tpw == 8) join(k_wjoin<8>);
            else join(k_wjoin<4>);
        }
        exclusive_scan(c, tcnt, ntiles, toff, s);
        launch(c, "k_wsurv", 48.0 * nq, k_wsurv, wblocks(nq), WT, (const WQ *)d_q, nq, (const uint64_t *)F,
               (const uint64_t *)bitmap, (const uint32_t *)rec_r, (const uint64_t *)trow, ntiles, group,
               (const uint64_t *)toff, gba, sb);
        std::vector<uint64_t> hsb;
        read_words(c, sb, hsb, 4ull * nq);
        const uint64_t Stot = hsb[4ull * (nq - 1) + 1];
        // next tables (exact sizes) and result rows
        bool any_final = false;
        double kb = (recs ? 8.0 * Stot : gba / 8.0) + 8.0 * ntiles;
        for (uint32_t a = 0; a < nq; a++) {
            WideQuery &x = *act[a];
            WQ &Q = hq[a];
            Q.sbase = hsb[4 * a];
            Q.S = hsb[4 * a + 1] - hsb[4 * a];
            x.stats_gba[x.j] = hsb[4 * a + 3] - hsb[4 * a + 2];
            x.stats_surv[x.j] = Q.S;
            if (Q.S == 0) continue;
            kb += (double)Q.S * (4.0 + 4.0 * Q.j);
            if (Q.final_level) {
                any_final = true;
                if (!count_only) {
                    Q.out = persist<uint32_t>(c, Q.S * Q.k, "result rows");
                    x.rows = Q.out;
                    kb += 4.0 * Q.k * Q.S;
                }
            } else {
                x.next = c->arena.alloc(4ull * (Q.j + 1) * Q.S, false);
                if (!x.next)
                    fail(GSI_E_NOMEM, "arena exhausted allocating %llu bytes for a next table",
                         (unsigned long long)(4ull * (Q.j + 1) * Q.S));
                Q.Mn = static_cast<uint32_t *>(x.next);
                kb += 4.0 * (Q.j + 1) * Q.S;
            }
        }
        uint64_t *acc = nullptr, *d_dig = nullptr;
        if (any_final) {
            acc = s.get<uint64_t>(2ull * WACC * nq, "digest accumulators");
            d_dig = s.get<uint64_t>(2ull * nq, "digests");
            fill_u64(c, acc, 0, 2ull * WACC * nq);
        }
        GSI_HIP(hipMemcpyAsync(d_q, hq.data(), sizeof(WQ) * nq, hipMemcpyHostToDevice, c->stream));
        if (recs && Stot) {
            const uint32_t nlt = wblocks(Stot);
            uint64_t *stile = s.get<uint64_t>((uint64_t)nlt + 1, "wide survivor groups");
            tile_rows(c, toff, ngroups, nlt, WT, stile);
            auto link = [&](auto kern) {
                launch(c, "k_wlink", kb, kern, nlt, WT, (const WQ *)d_q, (const uint32_t *)rowq,
                       (const uint64_t *)trow, (const uint64_t *)toff, (const uint64_t *)stile, group,
                       (const uint32_t *)rec_x, (const uint32_t *)rec_r, Stot,
                       reinterpret_cast<unsigned long long *>(acc));
            };
            if (any_final && !count_only) link(k_wlink<true>);
            else link(k_wlink<false>);
        } else if (Stot) {
            auto link = [&](auto kern) {
                launch(c, "k_wlink_bits", kb, kern, (uint32_t)ngroups, WT, (const WQ *)d_q, (const uint32_t *)rowq,
                       (const uint64_t *)F, (const uint64_t *)trow, ntiles,
                       (const uint32_t *)loc, (const uint64_t *)bitmap, (const uint64_t *)toff,
                       reinterpret_cast<unsigned long long *>(acc));
            };
            if (tpw == 1) link(k_wlink_bits<1>);
            else if (tpw == 2) link(k_wlink_bits<2>);
            else if (tpw == 8) link(k_wlink_bits<8>);
            else link(k_wlink_bits<4>);
        }
        std::vector<uint64_t> dig;
        if (any_final) {
            launch(c, "k_wdigest", 16.0 * WACC * nq, k_wdigest, wblocks(nq), WT, (const uint64_t *)acc, nq, d_dig);
            read_words(c, d_dig, dig, 2ull * nq);  // and the uploads are done
        } else {
            sync(c);  // uploads done
        }
        if (any_final)
            for (uint32_t a = 0; a < nq; a++)
                if (hq[a].final_level) {
                    act[a]->digest[0] += dig[2ull * a];
                    act[a]->digest[1] ^= dig[2ull * a + 1];
                }
        pend.commit = true;
        for (uint32_t a = 0; a < nq; a++) {
            WideQuery &x = *act[a];
            const WQ &Q = hq[a];
            if (Q.S == 0) {
                x.levels = x.j;
                x.finish_empty();
            } else if (Q.final_level) {
                x.count = Q.S;
                x.levels = x.j;
                x.release_table();
                x.done = true;
            } else {
                x.release_table();
                x.own = x.next;
                x.next = nullptr;
                x.M = Q.Mn;
                x.R = Q.S;
                x.j++;
            }
        }
    }
}

// Estimated scratch bytes of one step for a query (lookups, bounds, F, one
// slot per row for the bitmap and tiles, and a next table of the same rows).
static uint64_t step_bytes(const WideQuery &x) {
    const uint64_t ne = x.j;  // at most j linking edges
    return x.R * (8 * ne + 4 + 8 + 8) + 4096;
}

WideEngine::WideEngine(gsi_graph *g, bool count_only, bool tolerant, uint32_t tiles)
    : g_(g), count_only_(count_only), tolerant_(tolerant),
      tpw_(tiles == 1 || tiles == 2 || tiles == 8 ? tiles : WJ_TILES) {}

void WideEngine::add(WideQuery &&q) { qs_.push_back(std::move(q)); }

bool WideEngine::idle() const {
    for (auto &x : qs_)
        if (!x.done) return false;
    return true;
}

uint32_t WideEngine::step() {
    std::vector<WideQuery *> act;
    for (auto &x : qs_)
        if (!x.done) act.push_back(&x);
    if (act.empty()) return 0;
    // start with the queries whose estimated step scratch fits in half the
    // largest free block; halve on an arena failure
    gsi_ctx *c = g_->ctx;
    const uint64_t room = c->arena.largest_free() / 2;
    size_t n = 0;
    uint64_t est = 0;
    while (n < act.size() && (n == 0 || est + step_bytes(*act[n]) <= room)) est += step_bytes(*act[n++]);
    size_t skipped = 0;  // queries moved behind the others (tolerant engine)
    bool records = true, filter = true;
    for (;;) {
        std::vector<WideQuery *> part(act.begin(), act.begin() + n);
        try {
            wide_step(g_, part, count_only_, tpw_, records, filter);
            steps_++;
            break;
        } catch (const Fail &f) {
            if (f.st != GSI_E_NOMEM) throw;
            if (n == 1 && !filter && !tolerant_) {
                // the tables of the others may be what it lacks
                bool freed = false;
                for (size_t i = 1; i < act.size(); i++) freed |= act[i]->restart();
                if (!freed) throw;
                records = filter = true;
                clear_error();
                continue;
            }
            clear_error();
            if (n == 1 && filter) {
                // what the records took may be what the next table lacked,
                // then what the filtered lists took
                if (records) records = false;
                else filter = false;
                continue;
            }
            if (n > 1) {
                n = (n + 1) / 2;
                continue;
            }
            WideQuery *x = act.front();
            if (act.size() == 1 || skipped + 1 >= act.size()) {
                // nothing else holds step memory that could be waited for
                x->release_table();
                x->status = GSI_E_NOMEM;
                x->count = 0;
                x->levels = x->j;
                x->done = true;
                break;
            }
            act.erase(act.begin());
            act.push_back(x);
            skipped++;
            records = filter = true;
        }
    }
    uint32_t done = 0;
    for (auto *x : act) done += x->done;
    return done;
}

std::vector<WideQuery> WideEngine::take_done() {
    std::vector<WideQuery> out, keep;
    for (auto &x : qs_) (x.done ? out : keep).push_back(std::move(x));
    qs_ = std::move(keep);
    return out;
}

void wide_run(gsi_graph *g, std::vector<WideQuery> &wq, bool count_only, uint32_t tiles) {
    WideEngine e(g, count_only, false, tiles);
    for (auto &x : wq) e.add(std::move(x));
    while (!e.idle()) e.step();
    wq = e.take_done();
}

}  // namespace gsi
