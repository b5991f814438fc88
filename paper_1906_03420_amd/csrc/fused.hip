// Fused join levels for small tables: one 1024-thread workgroup runs the
// levels of Algorithm 3 (with Algorithm 4's pre-allocation) back to back,
// with F, the GBA keep bits and the survivor prefix sums in LDS, so a level
// costs no kernel launch and no host round trip.  The workgroup stops at the
// first level whose rows, slots (|GBA|) or survivors exceed its capacity and
// reports where; the caller finishes the query from that level with the
// per-level kernels.  The single-query kernel can share its larger levels
// among the workgroups of its launch (see Cluster).  Results are identical to the per-level path (same
// tests, same order: parent row, then ascending x).
#include <cstddef>
#include <cstring>
#include <type_traits>

#include "fused.h"
#include "join_device.h"

namespace gsi {

// exclusive prefix sum over v (one value per thread), total in *total
template <uint32_t FT>
__device__ __forceinline__ uint32_t wg_exclusive_sum(uint32_t v, uint32_t *s_w, uint32_t *total) {
    const uint32_t lane = lane_id(), w = threadIdx.x >> 6;
    uint32_t inc = wave_inclusive_sum(v);
    if (lane == 63) s_w[w] = inc;
    __syncthreads();
    uint32_t off = 0, tot = 0;
#pragma unroll
    for (uint32_t q = 0; q < FT / 64; q++) {
        uint32_t x = s_w[q];
        off += q < w ? x : 0u;
        tot += x;
    }
    __syncthreads();
    *total = tot;
    return off + inc - v;
}

// Rows of U slots at once: for each r, the largest i < R with F[i] <= p[r]
// (F in LDS, non-decreasing, F[0] = 0), with Fi[r] = F[i].  A branch-free
// binary lifting with the same number of steps for every lane, so the U
// searches interleave their LDS reads.  F[R] (|GBA|) is read in place of
// indices past the table; it exceeds every slot below |GBA|.
template <uint32_t U>
__device__ __forceinline__ void lds_rows(const uint32_t *F, uint32_t R, const uint32_t *p, uint32_t *row,
                                         uint32_t *Fi) {
#pragma unroll
    for (uint32_t r = 0; r < U; r++) {
        row[r] = 0;
        Fi[r] = 0;
    }
    for (uint32_t b = R > 1 ? 1u << (31 - __builtin_clz(R - 1)) : 0u; b; b >>= 1) {
#pragma unroll
        for (uint32_t r = 0; r < U; r++) {
            const uint32_t m = row[r] + b;
            const uint32_t f = F[m < R ? m : R];
            if (m < R && f <= p[r]) {
                row[r] = m;
                Fi[r] = f;
            }
        }
    }
}

// Position of the r-th set bit (r from 0) of m, which has more than r set bits.
__device__ __forceinline__ uint32_t nth_set_bit(uint64_t m, uint32_t r) {
    uint32_t pos = 0;
#pragma unroll
    for (uint32_t sh = 32; sh; sh >>= 1) {
        const uint32_t c = (uint32_t)__popcll(m & ((1ull << sh) - 1));
        if (r >= c) {
            r -= c;
            m >>= sh;
            pos += sh;
        }
    }
    return pos;
}

// For U survivors q[r] < S: the bitmap word holding each (the largest w <
// nw with pre[w] <= q, pre being the exclusive prefix of the words' set
// bits, in LDS) and the survivor's rank within it.  Branch-free, as lds_rows.
template <uint32_t U>
__device__ __forceinline__ void lds_words(const uint32_t *pre, uint32_t nw, const uint32_t *q, uint32_t *wd,
                                          uint32_t *rk) {
#pragma unroll
    for (uint32_t r = 0; r < U; r++) {
        wd[r] = 0;
        rk[r] = q[r];
    }
    for (uint32_t b = nw > 1 ? 1u << (31 - __builtin_clz(nw - 1)) : 0u; b; b >>= 1) {
#pragma unroll
        for (uint32_t r = 0; r < U; r++) {
            const uint32_t m = wd[r] + b;
            const uint32_t f = pre[m < nw ? m : nw - 1];
            if (m < nw && f <= q[r]) {
                wd[r] = m;
                rk[r] = q[r] - f;
            }
        }
    }
}

// s_waitcnt operand: vmcnt 0, the other counters unconstrained (gfx9 encoding)
constexpr int WAIT_VMCNT0 = 0x0F70;

// bitmap words a wave takes per round of the fused join and link, and per
// round of the candidate pass of a level of more than one round
constexpr uint32_t FU = 2, FP = 4;

// Words of each of the two LDS buffers that hold intermediate tables small
// enough (rows x columns), sized to what the workgroup's LDS has left.
template <uint32_t FT, bool XS>
constexpr uint32_t fused_table_words() {
    return FT == 1024 ? (XS ? 6912u : 14336u) : FT == 256 ? 1536u : 384u;
}

// LDS of one fused workgroup with FT threads, CR rows and CS slots: F, the
// start of each row's scanned list, the keep bits (and a second copy for
// the candidate pass) and their prefix sums,
// (XS) each slot's element x, so that the link re-reads no list, and two
// table buffers
//
// FusedStat: the words of an FStatus, its per-level sizes in 32 bits (|GBA| of
// a level that does not fit stops there; all others are below)
enum : uint32_t { ST_DONE, ST_LEVEL, ST_ROWS, ST_MLOC, ST_LEVELS, ST_COUNT, ST_DIG0, ST_DIG1, ST_OUT_BASE, FSTAT_HEAD };
struct FusedStat {
    uint64_t head[FSTAT_HEAD];
    uint32_t lv[3 * GSI_MAX_K];  // rows, |GBA| and survivors of each level
};
static_assert(sizeof(FStatus) == 8 * (FSTAT_HEAD + 3 * GSI_MAX_K) && offsetof(FStatus, lv_rows) == 8 * FSTAT_HEAD,
              "FusedStat lists the words of an FStatus");

template <uint32_t FT, uint32_t CR, uint32_t CS, bool XS>
struct FusedLds {
    FusedStat s;
    uint32_t F[CR + 1];
    uint32_t st[CR];
    uint64_t bits[CS / 64];
    uint64_t keep[CS / 64];
    uint32_t wpre[CS / 64];
    uint32_t w[FT / 64];
    uint64_t d[2][FT / 64];
    uint64_t obase;
    uint32_t x[XS ? CS : 1];
    uint32_t mt[2][fused_table_words<FT, XS>()];
};
// The single-query kernel's LDS: the workgroup's and a copy of the plan.
struct ClusterLds {
    uint64_t pre[CL_MAX_WG + 1];  // of the last meeting: the values before each workgroup's, and their sum
    uint32_t w[8];
};

struct FusedLevelsLds {
    FusedLds<1024, FUSED_MAX_ROWS, FUSED_MAX_SLOTS, true> q;
    FPlanArg plan;
    ClusterLds cl;
};
static_assert(sizeof(FusedLevelsLds) <= 160 * 1024, "fused workgroup LDS");

// A value every lane holds alike, in scalar registers.  No other type
// converts to one of these: a 64-bit sum must not lose its upper half.
__device__ __forceinline__ uint32_t uni(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ uint64_t uni(uint64_t v) {
    return ((uint64_t)uni((uint32_t)(v >> 32)) << 32) | uni((uint32_t)v);
}
template <typename T>
__device__ __forceinline__ T *uni(T *p) {
    return reinterpret_cast<T *>(uni(reinterpret_cast<uint64_t>(p)));
}
template <typename T>
void uni(T) = delete;

// What a workgroup reports of its query: kept in LDS while the levels run
// and written out once at the end (st_flush).  A store to the status inside
// a level costs its wave the acknowledgement at the next load it waits for,
// the more so when the status lies in host memory.
__device__ __forceinline__ void st_clear(FusedStat &s) {
    uint32_t *w = reinterpret_cast<uint32_t *>(&s);
    for (uint32_t t = threadIdx.x; t < sizeof(FusedStat) / 4; t += blockDim.x) w[t] = 0;
}
// the first wave writes `s` to `st`
__device__ __forceinline__ void st_flush(const FusedStat &s, FStatus *st) {
    if (threadIdx.x >= 64) return;
    for (uint32_t t = threadIdx.x; t < sizeof(FStatus) / 8; t += 64) {
        uint64_t v;
        if (t < FSTAT_HEAD) v = s.head[t];
        else v = s.lv[t - FSTAT_HEAD];
        reinterpret_cast<uint64_t *>(st)[t] = v;
    }
}

// ----------------------------------------------------------- cluster
// A level of a few thousand slots keeps one CU busy for tens of microseconds
// (a CU brings in some 300 scattered lines per microsecond) while the rest of
// the chip idles, and handing it to the per-level kernels costs five launches
// and a host round trip.  The single-query kernel is launched with further
// workgroups (helpers) that wait while the first one runs small levels alone;
// on a larger one it publishes the table, and it and the helpers locate equal
// parts of its rows and join those, or equal shares of all their slots, in
// order, so a level's rows come out in the same order.  The meeting points of
// a shared level are the parts' weights, (where the slots are dealt out anew)
// the rows' lists, the survivor counts, which give every workgroup its place
// in the next table, and the table's completion; 2 us each, 3 with fences.
// On 10^6 vertices 16 walk queries went from 3.79 to 3.5 ms, 8 homomorphism
// queries from 1.98 to 1.8 ms.
//
// Only helpers that have checked in are called, so no workgroup waits for one
// that is not running (another stream may hold the CUs).  Every wait is
// bounded all the same: past CL_SPINS polls a workgroup sets `abort` and
// leaves, the others see the flag and leave too, and the first reports that
// it stopped at the table it was given, which nothing has overwritten.
constexpr uint32_t CL_SPINS = 1u << 16;  // about 50 ms
constexpr uint32_t CL_HERE_SPINS = 16;   // about 10 us

// How long the workgroups wait and whether they are there: other values than
// these in tests only, by the context's flags.
struct ClusterWaits {
    uint32_t spins = CL_SPINS;  // polls after which a wait runs out
    uint32_t quit = 0;          // the meeting at which workgroup 1 leaves, or CL_ABSENT
};
constexpr uint32_t CL_ABSENT = 0xFFFFFFFFu;  // no helper checks in
static ClusterWaits cluster_waits(const gsi_ctx *c) {
    ClusterWaits w;
    if (c->flags & GSI_CTX_TEST_SHORT_WAITS) w.spins = 64;
    w.quit = c->flags & GSI_CTX_TEST_NO_HELPERS ? CL_ABSENT : (c->flags >> 16) & 255u;
    return w;
}

// One atomic word carries a workgroup's epoch and its value, so the values
// need no fence.  Two sets of words: a workgroup writes epoch e + 2 only after
// all have read epoch e.
struct ClusterCtl {
    unsigned long long word[2][CL_MAX_WG];
    unsigned long long call;   // the last call: its number << 32 | level << 8 | workgroups
    uint32_t here[CL_MAX_WG];  // helper checked in
    uint32_t abort;
    uint32_t args[4];          // of the last call: rows, stride, place, epoch
    unsigned long long dig[CL_MAX_WG][2];  // digests of a shared last level
};
static_assert(sizeof(ClusterCtl) <= CL_CTL_BYTES && CL_CTL_BYTES % 8 == 0, "control block");

struct Cluster {
    ClusterCtl *c;
    uint32_t bid;       // this workgroup among them
    uint32_t nmax;      // workgroups launched
    uint32_t nb;        // those of the last call
    uint32_t cap_rows;  // rows of a shared level's table
    uint32_t cap_out;   // result rows
    uint32_t epoch, call;
    ClusterWaits waits;
    ClusterLds *l;
};

template <typename T>
__device__ __forceinline__ T cl_load(const T *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void cl_store(T *p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// All workgroups meet: cl.l->pre gets the sums of `value` over the workgroups
// before each one, and over all of them at pre[nb], w[1] the largest.  With `table`, what every
// thread wrote before is visible to every workgroup after.  False when a wait
// ran out.  Called by all threads; a barrier must follow before the next one.
__device__ __forceinline__ bool cl_meet(Cluster &cl, bool table, uint32_t value) {
    const uint32_t e = ++cl.epoch;
    if (table) {
        __builtin_amdgcn_s_waitcnt(WAIT_VMCNT0);
        __syncthreads();
    }
    if (threadIdx.x < 64) {
        if (table) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        unsigned long long *w = cl.c->word[e & 1];
        const uint32_t lane = threadIdx.x;
        if (lane == 0) cl_store(w + cl.bid, ((unsigned long long)e << 32) | value);
        unsigned long long x = 0;
        bool ok = lane >= cl.nb, dead = cl.bid == 1 && e == cl.waits.quit;
        for (uint32_t spins = 1; !dead && __ballot(!ok); spins++) {
            if (!ok) {
                x = cl_load(w + lane);
                ok = (uint32_t)(x >> 32) == e;
            }
            if (spins > cl.waits.spins || ((spins & 63) == 0 && uni(cl_load(&cl.c->abort)))) {
                dead = true;
                break;
            }
        }
        if (dead && lane == 0) cl_store(&cl.c->abort, 1u);
        const uint64_t v = lane < cl.nb ? (uint64_t)(uint32_t)x : 0ull;
        uint64_t inc = v;
#pragma unroll
        for (uint32_t d = 1; d < 64; d *= 2) {
            const uint64_t o = __shfl_up(inc, d, 64);
            if (lane >= d) inc += o;
        }
        if (table) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        uint32_t most = (uint32_t)v;
#pragma unroll
        for (uint32_t d = 32; d; d /= 2) {
            const uint32_t o = __shfl_xor(most, d, 64);
            most = o > most ? o : most;
        }
        if (lane < cl.nb) cl.l->pre[lane + 1] = inc;
        if (lane == 0) {
            cl.l->pre[0] = 0;
            cl.l->w[0] = dead ? 1u : 0u;
            cl.l->w[1] = most;
        }
    }
    __syncthreads();
    return uni(cl.l->w[0]) == 0;
}

// The row of a shared level of R rows that holds weight a: the rows' weights
// before them are pre[c] (of their part c) plus W[row].  Called by a wave.
__device__ __forceinline__ uint32_t cl_row(const Cluster &cl, const uint32_t *W, uint32_t R, uint64_t a) {
    const uint32_t lane = threadIdx.x & 63;
    // the last part that starts at or before a and has rows
    const uint32_t nb = cl.nb;
    const uint32_t lo0 = (uint32_t)((uint64_t)R * lane / nb), hi0 = (uint32_t)((uint64_t)R * (lane + 1) / nb);
    const uint64_t in = __ballot(lane < nb && lo0 < hi0 && cl.l->pre[lane] <= a);
    const uint32_t c = in ? 63u - (uint32_t)__builtin_clzll(in) : 0u;
    uint32_t lo = uni((uint32_t)((uint64_t)R * c / nb));
    const uint32_t hi = uni((uint32_t)((uint64_t)R * (c + 1) / nb));
    const uint64_t rel = a - cl.l->pre[c];
    // 64 probes a round: row lo starts at or before a, row lo + n after it
    uint32_t n = hi > lo ? hi - lo : 1u;
    while (n > 1) {
        const uint32_t step = (n + 63) / 64;
        const uint32_t t = lane * step;
        const uint64_t le = __ballot(t < n && (uint64_t)W[lo + (t < n ? t : 0u)] <= rel);
        const uint32_t m = le ? 63u - (uint32_t)__builtin_clzll(le) : 0u;
        lo += m * step;
        n = n - m * step < step ? n - m * step : step;
    }
    return lo;
}

// The call of the first workgroup: level j of the table of R rows (stride
// ld) at `mloc`, at most `share` of them to a workgroup; j = 0 lets the
// helpers go.  Called by all its threads, with the table written.  False, and
// no call, when too few helpers have checked in.
//
// Level and workgroups are in the word that a helper polls, so one that is
// not called reads nothing that a later call may be writing; one that is
// called has read `args` before the first meeting, and the first workgroup
// does not write them again before it.
__device__ __forceinline__ bool cl_call(Cluster &cl, uint32_t j, uint32_t R, uint32_t ld, uint32_t mloc,
                                        uint32_t share) {
    __builtin_amdgcn_s_waitcnt(WAIT_VMCNT0);
    __syncthreads();
    if (threadIdx.x < 64) {
        const uint32_t lane = threadIdx.x;
        uint32_t nb = 1;
        for (uint32_t spins = 0;; spins++) {
            const bool here = lane == 0 || (lane < cl.nmax && cl_load(cl.c->here + lane) != 0);
            const uint64_t out = ~__ballot(here);
            nb = out ? (uint32_t)__builtin_ctzll(out) : 64u;  // the first ones in a row
            // the first call gives helpers that are just starting a moment
            if (j == 0 || cl.call || nb == cl.nmax || spins == CL_HERE_SPINS) break;
        }
        const bool ok = j == 0 || (nb > 1 && R <= nb * share);
        if (lane == 0) {
            cl.l->w[0] = ok ? nb : 0u;
            if (ok) {
                cl_store(cl.c->args, R);
                cl_store(cl.c->args + 1, ld);
                cl_store(cl.c->args + 2, mloc);
                cl_store(cl.c->args + 3, cl.epoch);
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
                cl_store(&cl.c->call, ((unsigned long long)(cl.call + 1) << 32) | (j << 8) | nb);
            }
        }
    }
    __syncthreads();
    const uint32_t nb = uni(cl.l->w[0]);
    __syncthreads();
    if (!nb) return false;
    cl.nb = nb;
    cl.call++;
    return true;
}

// A helper's wait for the next call that includes it; false when it is to
// leave.
__device__ __forceinline__ bool cl_wait(Cluster &cl, uint32_t *j, uint32_t *R, uint32_t *ld, uint32_t *mloc) {
    if (threadIdx.x < 64) {
        uint32_t lv = 0, nb = 0;
        bool dead = false;
        if (threadIdx.x == 0 && cl.waits.quit != CL_ABSENT) cl_store(cl.c->here + cl.bid, 1u);
        for (uint32_t spins = 1;; spins++) {
            const unsigned long long x = cl_load(&cl.c->call);
            const uint32_t n = uni((uint32_t)(x >> 32));
            lv = uni((uint32_t)x) >> 8;
            nb = uni((uint32_t)x) & 255u;
            if (n != cl.call && (lv == 0 || nb > cl.bid)) {
                cl.call = n;
                break;
            }
            if (spins > cl.waits.spins || ((spins & 63) == 0 && uni(cl_load(&cl.c->abort)))) {
                dead = true;
                break;
            }
            __builtin_amdgcn_s_sleep(8);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        if (dead && threadIdx.x == 0) cl_store(&cl.c->abort, 1u);
        if (threadIdx.x == 0) {
            cl.l->w[0] = dead ? 0u : lv;
            cl.l->w[1] = cl.call;
            cl.l->w[2] = nb;
#pragma unroll
            for (uint32_t t = 0; t < 4; t++) cl.l->w[t + 3] = cl_load(cl.c->args + t);
        }
    }
    __syncthreads();
    *j = uni(cl.l->w[0]);
    cl.call = uni(cl.l->w[1]);
    cl.nb = uni(cl.l->w[2]);
    *R = uni(cl.l->w[3]);
    *ld = uni(cl.l->w[4]);
    *mloc = uni(cl.l->w[5]);
    cl.epoch = uni(cl.l->w[6]);
    __syncthreads();
    return *j != 0;
}

// Join levels j0 .. k-1 of one query in one workgroup (see the file
// comment), starting from the table M0 of R0 rows and j0 columns (column c
// at M0 + c * ld0).  FT threads; at most CR rows per table (CR = 4 FT) and
// CS slots per level.  With `ocount` set, the last level reserves its S*k
// output words from that counter (words of `out`, at most `ocap`) instead of
// writing at out[0].  CL: the workgroups of `cl` share levels of more than
// CL_ROWS rows or CL_SLOTS slots (the first workgroup runs the others, and
// returns with the status); buf0 and buf1 then hold cl->cap_rows rows.
template <uint32_t FT, uint32_t CR, uint32_t CS, bool XS, bool CL = false>
__device__ __forceinline__ void fused_query(const FPlan *plan, uint32_t j0, const uint32_t *M0, uint32_t R0,
                                            uint32_t ld0, uint32_t *buf0, uint32_t *buf1, uint32_t *loc,
                                            uint32_t *out, FusedLds<FT, CR, CS, XS> &L,
                                            unsigned long long *ocount = nullptr, uint64_t ocap = 0,
                                            Cluster *cl = nullptr) {
    static_assert(CR == 4 * FT, "each thread scans four rows");
    static_assert(CS / 64 <= FT, "one thread per bitmap word in the survivor scan");
    uint32_t *s_F = L.F;
    uint64_t *s_bits = L.bits;
    uint32_t *s_wpre = L.wpre;
    uint32_t *s_w = L.w;

    const uint32_t tid = threadIdx.x, lane = lane_id(), w = tid >> 6;
    const uint32_t k = uni(plan->k);
    const uint32_t cap_rows = plan->cap_rows < CR ? plan->cap_rows : CR;
    const uint32_t cap_slots = plan->cap_slots < CS ? plan->cap_slots : CS;
    const uint32_t *M = M0;
    uint32_t R = R0;
    uint32_t ld = ld0;  // column stride of M
    uint32_t mloc = FSTATUS_IN_FIRST;  // where M lives
    // A table of at most MT words is written to (and read from) LDS instead
    // of global memory; M then has column stride R.  M sits at index
    // next ^ 1 of its space (global or LDS), M' goes to index `next`.
    constexpr uint32_t MT = fused_table_words<FT, XS>();
    constexpr uint32_t PAD = CL ? CL_ROW_WEIGHT : 0;
    static_assert(!CL || CS / PAD + 2 <= CR, "rows of a share");
    constexpr uint32_t SHARE_ROWS = CL ? CL_CAP_ROWS / CL_MAX_WG : CR;  // rows a workgroup locates
    static_assert(SHARE_ROWS <= CR && (!CL || (uint64_t)SHARE_ROWS * (CL_MAX_WG * CS + 1 + PAD) < (1ull << 32)),
                  "weights of the located rows");
    bool m_lds = false;
    uint32_t next = 0;
    const bool cluster = CL && cl->nmax > 1;
    const uint32_t bid = CL ? cl->bid : 0u;
    bool wide = false;  // the level is shared
    // level j does not fit: record where, and where its input M lives (a
    // table in LDS is copied to buf0 for the caller)
    auto stop = [&](uint32_t j) {
        if (m_lds) {
            for (uint32_t t = tid; t < R * j; t += FT) buf0[t] = M[t];
            mloc = 0;
        }
        if (tid == 0) {
            L.s.head[ST_LEVEL] = j;
            L.s.head[ST_ROWS] = R;
            L.s.head[ST_MLOC] = mloc;
        }
    };
    if (R0 > (cluster ? cl->cap_rows : cap_rows)) {  // the first table does not fit
        stop(j0);
        return;
    }
    // the first workgroup calls the helpers to level j (a table in LDS is
    // written to buf0 for them); once per level, for none may be there
    uint32_t called = 0;
    auto go_wide = [&](uint32_t j) {
        called = j;
        if (m_lds) {
            for (uint32_t t = tid; t < R * j; t += FT) buf0[t] = M[t];
            M = buf0;
            m_lds = false;
            mloc = 0;
        }
        wide = cl_call(*cl, j, R, ld, mloc, SHARE_ROWS);
        next = mloc == 0 ? 1u : 0u;
    };
    // a wait ran out: the query starts over from its first table
    auto give_up = [&]() {
        if (tid == 0) {
            L.s.head[ST_LEVEL] = j0;
            L.s.head[ST_ROWS] = R0;
            L.s.head[ST_MLOC] = FSTATUS_IN_FIRST;
        }
    };

    for (uint32_t j = j0; j < k; j++) {
        if (cluster && !wide) {
            if (bid != 0) {
                if (!cl_wait(*cl, &j, &R, &ld, &mloc)) return;
                M = mloc == FSTATUS_IN_FIRST ? M0 : mloc ? buf1 : buf0;
                wide = true;
                next = mloc == 0 ? 1u : 0u;
            } else if (R > CL_ROWS && called != j) {
                go_wide(j);
            }
            if (!wide && R > cap_rows) {
                stop(j);
                return;
            }
        }
        // the workgroup's rows of the table: Rw of them from row r0 (all but
        // when the level is shared), lookups of stride ls
        uint32_t r0 = wide ? (uint32_t)((uint64_t)R * bid / cl->nb) : 0u;
        uint32_t Rw = wide ? (uint32_t)((uint64_t)R * (bid + 1) / cl->nb) - r0 : R;
        const uint32_t ls = R;
        // a longer list does not fit whatever the others are
        const uint32_t max_bound = (wide ? cl->nb * CS : CS) + 1;
        const uint32_t ne = uni(plan->lv_ne[j]), ef = uni(plan->lv_first[j]), e0 = uni(plan->lv_e0[j]);
        const uint64_t *Cu = uni(plan->Cu[j]);
        const bool final_level = (j == k - 1);
        const uint32_t *ci_all = uni(plan->ci_all);
        const uint32_t lv_mmask = uni(plan->lv_mmask[j]);
        const bool homo = uni(plan->homo) != 0;
        if (tid == 0) L.s.lv[j] = R;

        // locate N(v, l) for every row and linking edge; the row scans the
        // list of e0 (Algorithm 4) or, with `pick`, its shortest one
        for (uint32_t i = tid; i < Rw; i += FT) {
            uint32_t s0 = 0, l0 = 0, ob = NONE32, os = 0, ol = 0xFFFFFFFFu;
            for (uint32_t e = 0; e < ne; e++) {
                const FEdge &ed = plan->edges[ef + e];
                const uint32_t v = M[(uint64_t)uni(ed.col) * ld + r0 + i];
                const uint2 r = pcsr_find(uni(ed.gl), uni(ed.G), uni(ed.H), v);
                reinterpret_cast<uint2 *>(loc)[(uint64_t)e * ls + r0 + i] = r;
                if (e == e0) {
                    s0 = r.x;
                    l0 = r.y;
                } else if (r.y < ol) {
                    ob = e;
                    os = r.x;
                    ol = r.y;
                }
            }
            uint32_t be = e0, bs = s0, bl = l0;
            if (plan->pick && ob != NONE32 && ol < l0) {
                be = ob;
                bs = os;
                bl = ol;
            }
            s_F[i] = (bl < max_bound ? bl : max_bound) + (wide ? PAD : 0u);
            L.st[i] = plan->edges[ef + be].ci_off + bs;
            if (ne > 1) loc[(uint64_t)(2 * ne) * ls + r0 + i] = be;
        }
        __syncthreads();
        // F = exclusive prefix sum of the bounds (each thread owns 4 rows)
        auto scan_F = [&]() {
            uint32_t v4[4], sum = 0;
#pragma unroll
            for (int q = 0; q < 4; q++) {
                uint32_t i = 4 * tid + q;
                v4[q] = i < Rw ? s_F[i] : 0u;
                sum += v4[q];
            }
            uint32_t tot;
            uint32_t run = wg_exclusive_sum<FT>(sum, s_w, &tot);
#pragma unroll
            for (int q = 0; q < 4; q++) {
                uint32_t i = 4 * tid + q;
                if (i < Rw) s_F[i] = run;
                run += v4[q];
            }
            if (tid == 0) s_F[Rw] = tot;
            __syncthreads();
        };
        scan_F();
        if (wide) {
            // every part's weight
            const uint32_t weight = uni(s_F[Rw]);
            if (!cl_meet(*cl, false, weight)) {
                give_up();
                return;
            }
            const uint32_t nb = cl->nb;
            // a part's weight is below 2^32, their sum is not
            const uint64_t T = uni(cl->l->pre[nb]);
            const uint64_t slots = T - (uint64_t)PAD * R;
            if (tid == 0) L.s.lv[GSI_MAX_K + j] = slots < NONE32 ? (uint32_t)slots : NONE32;
            if (T > (uint64_t)nb * CS) {
                stop(j);
                return;
            }
            if (T == (uint64_t)PAD * R) {  // no slots
                if (tid == 0) {
                    L.s.lv[2 * GSI_MAX_K + j] = 0;
                    L.s.head[ST_LEVELS] = j;
                    L.s.head[ST_DONE] = 1;
                }
                return;
            }
            // Parts differ: rows that follow each other often share a parent,
            // a hub's list is in all of them, and the largest part was 4 to
            // 10 times the mean on power-law graphs.  Where it is large, each
            // workgroup takes an equal share of the weight instead, cut
            // inside a row where it falls there.
            if (uni(cl->l->w[1]) <= CL_EVEN) {
                // the parts as they are; the padding goes
                static_assert(!CL || CL_EVEN / CL_ROW_WEIGHT < FT, "rows of a part");
                const uint32_t f = s_F[tid <= Rw ? tid : 0u];
                __syncthreads();
                if (tid <= Rw) s_F[tid] = f - PAD * tid;
            } else {
                uint32_t *gW = loc + (uint64_t)(2 * ne + 1) * ls, *gS = gW + ls, *gL = gS + ls;
                for (uint32_t i = tid; i < Rw; i += FT) {
                    const uint32_t f = s_F[i];
                    gW[r0 + i] = f;
                    gS[r0 + i] = L.st[i];
                    gL[r0 + i] = s_F[i + 1] - f - PAD;
                }
                if (!cl_meet(*cl, true, weight)) {
                    give_up();
                    return;
                }
                const uint32_t wa = (uint32_t)(T * bid / nb), wb = (uint32_t)(T * (bid + 1) / nb);
                if (w < 2) {
                    const uint32_t r = wa == wb ? 0u : cl_row(*cl, gW, R, w ? wb - 1 : wa);
                    if (lane == 0) cl->l->w[2 + w] = r;
                }
                __syncthreads();
                r0 = uni(cl->l->w[2]);
                Rw = wa == wb ? 0u : uni(cl->l->w[3]) + 1 - r0;
                for (uint32_t i = tid; i < Rw; i += FT) {
                    const uint32_t c = (uint32_t)(((uint64_t)(r0 + i + 1) * nb - 1) / R);  // the row's part
                    const uint32_t wr = (uint32_t)cl->l->pre[c] + gW[r0 + i], len = gL[r0 + i];
                    const uint32_t lo = wr > wa ? wr : wa, hi = wr + len < wb ? wr + len : wb;
                    s_F[i] = hi > lo ? hi - lo : 0u;
                    L.st[i] = gS[r0 + i] + (lo - wr);
                }
                __syncthreads();
                scan_F();
            }
            __syncthreads();
        }
        const uint32_t *Mw = M + r0;
        // values every thread reads from LDS are made wave-uniform, so that
        // the exits below are uniform branches
        const uint32_t gba = __builtin_amdgcn_readfirstlane(s_F[Rw]);
        if (tid == 0 && !wide) L.s.lv[GSI_MAX_K + j] = gba;
        if (cluster && !wide && gba > CL_SLOTS && called != j) {
            go_wide(j);
            j--;  // the level again, shared (or alone)
            continue;
        }
        if (!wide && gba > cap_slots) {
            // what the level does hold, for who runs it next: the lists' full
            // lengths (each thread reads the rows that it located)
            uint64_t sum = 0;
            for (uint32_t i = tid; i < R; i += FT)
                sum += reinterpret_cast<const uint2 *>(loc)[(uint64_t)(ne > 1 ? loc[(uint64_t)(2 * ne) * ls + i] : 0u) * ls + i].y;
            sum = wave_sum(sum);
            if (lane == 0) L.d[0][w] = sum;
            __syncthreads();
            if (tid == 0) {
                uint64_t all = 0;
                for (uint32_t q = 0; q < FT / 64; q++) all += L.d[0][q];
                L.s.lv[GSI_MAX_K + j] = all < NONE32 ? (uint32_t)all : NONE32;
            }
            stop(j);
            return;
        }
        if (!wide && gba == 0) {
            if (tid == 0) {
                L.s.lv[2 * GSI_MAX_K + j] = 0;
                L.s.head[ST_LEVELS] = j;
                L.s.head[ST_DONE] = 1;
            }
            return;
        }
        const uint32_t nw = (gba + 63) / 64;

        // join: keep x = N(v'_i, l0)[p - F[i]] iff x not in m_i, x in C(u),
        // x in every other linking list; one ballot word per 64 slots.  A
        // wave takes several words per round (words base + r * waves + w)
        // and issues each step's loads for all of them together, so a round
        // costs one chain of dependent loads.
        //
        // the tests after C(u), for U slots of rows ir
        const bool more_tests = (!homo && lv_mmask) || ne > 1;
        auto tests = [&](auto U_, const uint32_t *xr, const uint32_t *ir, bool *kp) {
            constexpr uint32_t U = decltype(U_)::value;
            if (!homo) {
                // x not among the row's values in the columns that can hold
                // it (those of u's label), four columns at a time; past the
                // last one the last is read again
                uint32_t mm = lv_mmask;
                const uint32_t last = mm ? 31u - (uint32_t)__builtin_clz(mm) : 0u;
                while (mm) {
                    uint32_t cq[4];
#pragma unroll
                    for (uint32_t q = 0; q < 4; q++) {
                        cq[q] = mm ? (uint32_t)__builtin_ctz(mm) : last;
                        mm &= mm - 1;
                    }
                    uint32_t mv[U][4];
#pragma unroll
                    for (uint32_t r = 0; r < U; r++)
#pragma unroll
                        for (uint32_t q = 0; q < 4; q++) mv[r][q] = Mw[(uint64_t)cq[q] * ld + ir[r]];
#pragma unroll
                    for (uint32_t r = 0; r < U; r++)
#pragma unroll
                        for (uint32_t q = 0; q < 4; q++) kp[r] = kp[r] && mv[r][q] != xr[r];
                }
            }
            if (ne < 2) return;
            uint32_t be[U];
#pragma unroll
            for (uint32_t r = 0; r < U; r++) be[r] = loc[(uint64_t)(2 * ne) * ls + r0 + ir[r]];
            for (uint32_t e = 0; e < ne; e++) {
                uint32_t st[U], len[U];
                bool act[U], hit[U], any = false;
#pragma unroll
                for (uint32_t r = 0; r < U; r++) {
                    act[r] = kp[r] && e != be[r];
                    any |= act[r];
                }
                if (!any) continue;
#pragma unroll
                for (uint32_t r = 0; r < U; r++) {
                    const uint2 sl = reinterpret_cast<const uint2 *>(loc)[(uint64_t)e * ls + r0 + ir[r]];
                    st[r] = sl.x;
                    len[r] = act[r] ? sl.y : 0u;
                }
                in_sorted_many<U, true, 4>(uni(plan->edges[ef + e].ci), st, len, xr, hit);
#pragma unroll
                for (uint32_t r = 0; r < U; r++)
                    if (act[r]) kp[r] = hit[r];
            }
        };
        // U words per wave and round: the slots' elements (kept in L.x with
        // XS), C(u), and with `all` the other tests.  Loads are issued
        // unconditionally, a slot past |GBA| reading valid addresses (element
        // 0, row 0, column j - 1), and masked afterwards: a load behind a
        // branch waits for the one before.
        auto pass = [&](auto U_, bool all) {
            constexpr uint32_t U = decltype(U_)::value;
            for (uint32_t base = 0; base < nw; base += U * (FT / 64)) {
                uint32_t pr[U], ir[U], fr[U], xr[U];
                bool kp[U];
#pragma unroll
                for (uint32_t r = 0; r < U; r++) {
                    pr[r] = (base + r * (FT / 64) + w) * 64 + lane;
                    kp[r] = pr[r] < gba;
                }
                lds_rows<U>(s_F, Rw, pr, ir, fr);
#pragma unroll
                for (uint32_t r = 0; r < U; r++) {
                    if (!kp[r]) ir[r] = 0;
                    xr[r] = ci_all[kp[r] ? L.st[ir[r]] + (pr[r] - fr[r]) : 0u];
                    if (!kp[r]) xr[r] = 0;
                }
                {
                    uint64_t cw[U];
#pragma unroll
                    for (uint32_t r = 0; r < U; r++) cw[r] = Cu[xr[r] >> 6];
#pragma unroll
                    for (uint32_t r = 0; r < U; r++) {
                        if (XS && kp[r]) L.x[pr[r]] = xr[r];
                        kp[r] = kp[r] && ((cw[r] >> (xr[r] & 63)) & 1ull);
                    }
                }
                if (all) tests(U_, xr, ir, kp);
#pragma unroll
                for (uint32_t r = 0; r < U; r++) {
                    const uint64_t mask = __ballot(kp[r]);
                    const uint32_t word = base + r * (FT / 64) + w;
                    if (lane == 0 && word < nw) s_bits[word] = mask;
                }
            }
        };
        if (nw <= FU * (FT / 64)) {
            pass(std::integral_constant<uint32_t, FU>(), more_tests);
        } else {
            // more than one round: first C(u) alone, twice as many words in
            // flight, then the other tests on the slots that passed, in
            // dense waves (a round of both, chained, took 3 us whatever few
            // of its slots needed the second part)
            pass(std::integral_constant<uint32_t, FP>(), false);
            if (more_tests) {
                __syncthreads();
                uint32_t C;
                const uint64_t word = tid < nw ? s_bits[tid] : 0ull;
                const uint32_t ex = wg_exclusive_sum<FT>((uint32_t)__popcll(word), s_w, &C);
                C = uni(C);
                if (tid < nw) {
                    s_wpre[tid] = ex;
                    L.keep[tid] = word;
                }
                __syncthreads();
                for (uint32_t base = 0; base < C; base += FU * FT) {
                    uint32_t q[FU], wd[FU], rk[FU], pr[FU], ir[FU], fr[FU], xr[FU];
                    bool kp[FU];
#pragma unroll
                    for (uint32_t r = 0; r < FU; r++) {
                        q[r] = base + r * FT + tid;
                        kp[r] = q[r] < C;
                    }
                    lds_words<FU>(s_wpre, nw, q, wd, rk);
#pragma unroll
                    for (uint32_t r = 0; r < FU; r++)
                        pr[r] = kp[r] ? wd[r] * 64 + nth_set_bit(s_bits[wd[r]], rk[r]) : 0u;
                    lds_rows<FU>(s_F, Rw, pr, ir, fr);
#pragma unroll
                    for (uint32_t r = 0; r < FU; r++) {
                        if (!kp[r]) ir[r] = 0;
                        if (XS) xr[r] = L.x[pr[r]];
                        else xr[r] = ci_all[kp[r] ? L.st[ir[r]] + (pr[r] - fr[r]) : 0u];
                    }
                    tests(std::integral_constant<uint32_t, FU>(), xr, ir, kp);
#pragma unroll
                    for (uint32_t r = 0; r < FU; r++)
                        if (!kp[r] && q[r] < C) atomicAnd(&L.keep[pr[r] >> 6], ~(1ull << (pr[r] & 63)));
                }
                __syncthreads();
                if (tid < nw) s_bits[tid] = L.keep[tid];
            }
        }
        __syncthreads();
        // survivor positions: prefix sum of the words' popcounts
        uint32_t S;
        {
            uint32_t c = tid < nw ? (uint32_t)__popcll(s_bits[tid]) : 0u;
            uint32_t ex = wg_exclusive_sum<FT>(c, s_w, &S);
            S = __builtin_amdgcn_readfirstlane(S);
            if (tid < nw) s_wpre[tid] = ex;
            __syncthreads();
        }
        // the level's survivors, and this workgroup's place among them
        uint32_t off = 0, St = S;
        if (wide) {
            if (!cl_meet(*cl, false, S)) {
                give_up();
                return;
            }
            off = (uint32_t)uni(cl->l->pre[bid]);
            St = (uint32_t)uni(cl->l->pre[cl->nb]);
            const uint32_t next_cap = cl->nb * SHARE_ROWS < cl->cap_rows ? cl->nb * SHARE_ROWS : cl->cap_rows;
            if (tid == 0) L.s.lv[2 * GSI_MAX_K + j] = St;
            if (St > (final_level ? (plan->count_only ? 0xFFFFFFFFu : cl->cap_out) : next_cap)) {
                stop(j);
                return;
            }
        }
        if (tid == 0) L.s.lv[2 * GSI_MAX_K + j] = St;
        if (St == 0) {
            if (tid == 0) {
                L.s.head[ST_LEVELS] = j;
                L.s.head[ST_DONE] = 1;
            }
            return;
        }
        if (!wide && !final_level && S > cap_rows) {
            if (cluster && called != j) {
                go_wide(j);
                j--;  // the level again, shared: its table may be larger
                continue;
            }
            stop(j);
            return;
        }

        // a chunk reserves its output rows
        if (final_level && ocount && !plan->count_only) {
            if (tid == 0) {
                const unsigned long long need = (unsigned long long)S * k;
                const unsigned long long b = atomicAdd(ocount, need);
                L.obase = (b + need <= ocap) ? (uint64_t)b : ~0ull;
            }
            __syncthreads();
            const uint64_t lb = L.obase;
            const uint64_t b = ((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(lb >> 32)) << 32) |
                               __builtin_amdgcn_readfirstlane((uint32_t)lb);
            if (b == ~0ull) {
                stop(j);
                return;
            }
            out += b;
            if (tid == 0) L.s.head[ST_OUT_BASE] = b;
        }

        // link: (m_i, x) at its position; the last level writes rows in
        // query-vertex order and hashes them.  Threads take survivors, not
        // slots (survivor q is at position q; its slot is found from the
        // keep bits' prefix sums), so the waves are dense however sparse the
        // keep bits are; FU survivors per thread and round.
        const bool n_lds = !wide && !final_level && (uint64_t)S * (j + 1) <= MT;
        // (selects, not an indexed pointer array, which would live in scratch)
        uint32_t *Mn = n_lds ? (next ? L.mt[1] : L.mt[0]) : (next ? buf1 : buf0);
        uint64_t hs = 0, hx = 0;
        for (uint32_t base = 0; base < S; base += FU * FT) {
            uint32_t pr[FU], ir[FU], fr[FU], pos[FU], xr[FU], wd[FU], rk[FU];
            bool kp[FU];
#pragma unroll
            for (uint32_t r = 0; r < FU; r++) {
                pos[r] = base + r * FT + tid;
                kp[r] = pos[r] < S;
            }
            lds_words<FU>(s_wpre, nw, pos, wd, rk);
#pragma unroll
            for (uint32_t r = 0; r < FU; r++) pr[r] = kp[r] ? wd[r] * 64 + nth_set_bit(s_bits[wd[r]], rk[r]) : 0u;
            lds_rows<FU>(s_F, Rw, pr, ir, fr);
            // unconditional loads from valid addresses, masked afterwards
#pragma unroll
            for (uint32_t r = 0; r < FU; r++) {
                if (!kp[r]) ir[r] = 0;
                if (XS) xr[r] = L.x[kp[r] ? pr[r] : 0u];
                else xr[r] = ci_all[kp[r] ? L.st[ir[r]] + (pr[r] - fr[r]) : 0u];
                if (!kp[r]) xr[r] = 0;
            }
            if (!final_level) {
                for (uint32_t c = 0; c < j; c += 4) {
                    uint32_t mv[FU][4];
#pragma unroll
                    for (uint32_t r = 0; r < FU; r++)
#pragma unroll
                        for (uint32_t q = 0; q < 4; q++)
                            mv[r][q] = Mw[(uint64_t)(c + q < j ? c + q : j - 1) * ld + ir[r]];
#pragma unroll
                    for (uint32_t r = 0; r < FU; r++)
#pragma unroll
                        for (uint32_t q = 0; q < 4; q++)
                            if (kp[r] && c + q < j) Mn[(uint64_t)(c + q) * St + off + pos[r]] = mv[r][q];
                }
#pragma unroll
                for (uint32_t r = 0; r < FU; r++)
                    if (kp[r]) Mn[(uint64_t)j * St + off + pos[r]] = xr[r];
            } else {
                uint64_t f[FU];
#pragma unroll
                for (uint32_t r = 0; r < FU; r++) f[r] = 14695981039346656037ull;
                for (uint32_t u0 = 0; u0 < k; u0 += 4) {
                    uint32_t val[FU][4];
#pragma unroll
                    for (uint32_t q = 0; q < 4; q++) {
                        const uint32_t c = u0 + q < k ? uni(plan->qcol[u0 + q]) : j;
#pragma unroll
                        for (uint32_t r = 0; r < FU; r++) {
                            const uint32_t mv = Mw[(uint64_t)(c < j ? c : 0u) * ld + ir[r]];
                            val[r][q] = c < j ? mv : xr[r];
                        }
                    }
#pragma unroll
                    for (uint32_t q = 0; q < 4; q++)
#pragma unroll
                        for (uint32_t r = 0; r < FU; r++) {
                            if (!kp[r] || u0 + q >= k) continue;
                            if (!plan->count_only) out[(uint64_t)(off + pos[r]) * k + u0 + q] = val[r][q];
                            f[r] = fnv_word(f[r], val[r][q]);
                        }
                }
#pragma unroll
                for (uint32_t r = 0; r < FU; r++) {
                    if (!kp[r]) continue;
                    const uint64_t h = mix64(f[r]);
                    hs += h;
                    hx ^= h;
                }
            }
        }
        if (final_level) {
            hs = wave_sum(hs);
            hx = wave_xor(hx);
            if (lane == 0) {
                L.d[0][w] = hs;
                L.d[1][w] = hx;
            }
            __syncthreads();
            if (tid == 0) {
                uint64_t ts = 0, tx = 0;
                for (uint32_t q = 0; q < FT / 64; q++) {
                    ts += L.d[0][q];
                    tx ^= L.d[1][q];
                }
                L.s.head[ST_DIG0] = ts;
                L.s.head[ST_DIG1] = tx;
                L.s.head[ST_COUNT] = St;
                L.s.head[ST_LEVELS] = j;
                if (!wide) {
                    L.s.head[ST_DONE] = 1;
                } else {
                    cl->c->dig[bid][0] = ts;
                    cl->c->dig[bid][1] = tx;
                }
            }
            if (wide) {
                if (!cl_meet(*cl, true, 0)) {
                    give_up();
                    return;
                }
                if (tid < 64) {
                    const uint64_t ts = wave_sum(tid < cl->nb ? (uint64_t)cl->c->dig[tid][0] : 0ull);
                    const uint64_t tx = wave_xor(tid < cl->nb ? (uint64_t)cl->c->dig[tid][1] : 0ull);
                    if (tid == 0) {
                        L.s.head[ST_DIG0] = ts;
                        L.s.head[ST_DIG1] = tx;
                        L.s.head[ST_DONE] = 1;
                    }
                }
            }
            return;
        }
        // M' complete before it is read as M
        if (wide) {
            if (!cl_meet(*cl, true, 0)) {
                give_up();
                return;
            }
            wide = St > CL_ROWS;
        } else {
            __syncthreads();
        }
        M = Mn;
        R = St;
        ld = St;
        m_lds = n_lds;
        if (!n_lds) mloc = next;
        next ^= 1u;
    }
}

// One query in one workgroup.  When `b0` is given, the first table M0 = C(u_first) is
// written here too from its bitset (ascending vertex order, R0 entries):
// each thread counts the set bits of a run of bitset words, an exclusive
// scan over the workgroup places the runs, and each thread writes its ids.
// INL: the plan is the kernel argument `inl`, copied to LDS first (the
// argument segment is read from host memory, a round trip of its own for
// every line the levels touch); else d_plan in device memory.  Two
// instances, not a select: a pointer that may address either space is
// generic.  Workgroups after the first help with its larger levels.
// At the end the status goes to `st` in one go and the completion word is
// posted (post_seq) once every wave's rows and tables have left it.
// CL: there are such workgroups (an instance of its own: what sharing adds to
// a level alone cost 0.4 us of 7).
template <bool INL, bool CL>
__global__ __launch_bounds__(1024) void k_fused_levels(const FPlan *d_plan, FPlanArg inl, uint32_t j0, uint32_t *M0,
                                                      uint32_t R0, const uint32_t *b0_runs,
                                                      const uint64_t *b0, uint64_t nwords, uint32_t *buf0,
                                                      uint32_t *buf1, uint32_t *loc, uint32_t *out, FStatus *st,
                                                      uint64_t *seq_slot, uint64_t seq_value, ClusterCtl *ctl,
                                                      uint32_t cl_rows, uint32_t cl_out, ClusterWaits waits) {
    __shared__ FusedLevelsLds L;
    const FPlan *plan = INL ? &L.plan.p : d_plan;
    if (INL) {
        static_assert(sizeof(FPlanArg) / 4 <= 1024, "one word per thread");
        if (threadIdx.x < sizeof(FPlanArg) / 4)
            reinterpret_cast<uint32_t *>(&L.plan)[threadIdx.x] = reinterpret_cast<const uint32_t *>(&inl)[threadIdx.x];
    }
    st_clear(L.q.s);
    if (b0 && blockIdx.x == 0) {
        // each wave owns a contiguous run of words (the split the filter's
        // counts used, whose per-run set bits `b0_runs` give the wave its
        // first output row), read 64 at a time (coalesced) with eight such
        // reads in flight, and emits with wave scans
        const uint32_t lane = lane_id(), wv = threadIdx.x >> 6;
        const uint64_t per = (nwords + BITS_RUNS - 1) / BITS_RUNS;
        const uint64_t ws = per * wv < nwords ? per * wv : nwords;
        const uint64_t we = ws + per < nwords ? ws + per : nwords;
        uint32_t at = wave_sum(lane < wv ? b0_runs[lane] : 0u);
        for (uint64_t base = ws; base < we; base += 512) {
            uint64_t m[8];
#pragma unroll
            for (uint32_t t = 0; t < 8; t++) {
                const uint64_t qq = base + 64 * t + lane;
                m[t] = qq < we ? b0[qq] : 0ull;
            }
#pragma unroll
            for (uint32_t t = 0; t < 8; t++) {
                const uint32_t pc = (uint32_t)__popcll(m[t]);
                const uint32_t inc = wave_inclusive_sum(pc);
                uint32_t o = at + inc - pc;
                uint64_t mm = m[t];
                const uint64_t qq = base + 64 * t + lane;
                while (mm) {
                    const uint32_t b = (uint32_t)__builtin_ctzll(mm);
                    if (o < R0) M0[o] = (uint32_t)(qq * 64 + b);
                    o++;
                    mm &= mm - 1;
                }
                at += __shfl(inc, 63, 64);
            }
        }
    }
    __syncthreads();  // status cleared, plan copied and M0 written before the levels read them
    Cluster cl{ctl, blockIdx.x, gridDim.x, 1u, cl_rows, cl_out, 0u, 0u, waits, &L.cl};
    fused_query<1024, FUSED_MAX_ROWS, FUSED_MAX_SLOTS, true, CL>(plan, j0, M0, R0, R0, buf0, buf1, loc, out, L.q,
                                                                 nullptr, 0, CL ? &cl : nullptr);
    if (blockIdx.x != 0) return;
    // every wave's stores are done before the first one releases them
    __builtin_amdgcn_s_waitcnt(WAIT_VMCNT0);
    __syncthreads();
    st_flush(L.q.s, st);
    if (threadIdx.x == 0) post_seq(seq_slot, seq_value);
    if (CL) cl_call(cl, 0, 0, 0, 0, 0);  // the helpers leave
}

void launch_fused(gsi_ctx *c, const FPlan *d_plan, const FPlanArg &inl, uint32_t j0, uint32_t *M0, uint32_t R0,
                  const uint32_t *b0_runs, const uint64_t *b0, uint64_t nwords, uint32_t *buf0, uint32_t *buf1, uint32_t *loc, uint32_t *out,
                  FStatus *d_status, double alg_bytes, const FusedCluster &fc) {
    uint64_t seqv = 0;
    uint64_t *seqp = seq_slot(c, d_status, &seqv);
    const auto go = [&](auto kernel) {
        launch(c, "k_fused_levels", alg_bytes, kernel, fc.nb, 1024, d_plan, inl, j0, M0, R0, b0_runs, b0, nwords, buf0,
               buf1, loc, out, d_status, seqp, seqv, reinterpret_cast<ClusterCtl *>(fc.ctl), fc.cap_rows, fc.cap_out,
               cluster_waits(c));
    };
    if (fc.nb > 1) {
        if (d_plan) go(k_fused_levels<false, true>);
        else go(k_fused_levels<true, true>);
    } else {
        if (d_plan) go(k_fused_levels<false, false>);
        else go(k_fused_levels<true, false>);
    }
    c->seq_armed = seqp != nullptr;
}

// Persistent batch: each workgroup takes the next query from a shared
// counter until none is left (every workgroup leaves once the counter passes
// the item count), and runs all its levels in its own scratch slot.
template <uint32_t FT, uint32_t CR, uint32_t CS>
// (the 256-thread tier is held to four waves per SIMD: left alone the
// compiler takes a few more registers and one workgroup per CU fewer fits)
__global__ __launch_bounds__(FT, FT == 256 ? 4 : 1) void k_fused_batch(const uint8_t *plans, const FBatchItem *items, uint32_t nitems,
                                                   const uint32_t *M0all, uint32_t *scratch, uint64_t slot_words,
                                                   uint32_t kmax, uint32_t *outall, FStatus *sts,
                                                   uint32_t *counter) {
    __shared__ FusedLds<FT, CR, CS, false> L;
    __shared__ uint32_t s_q;
    uint32_t *slot = scratch + (uint64_t)blockIdx.x * slot_words;
    uint32_t *buf0 = slot, *buf1 = slot + (uint64_t)CR * kmax, *loc = slot + 2ull * CR * kmax;
    for (;;) {
        if (threadIdx.x == 0) s_q = atomicAdd(counter, 1u);
        st_clear(L.s);
        __syncthreads();
        const uint32_t qi = __builtin_amdgcn_readfirstlane(s_q);
        __syncthreads();
        if (qi >= nitems) break;
        const FBatchItem it = items[qi];
        fused_query<FT, CR, CS, false>(reinterpret_cast<const FPlan *>(plans + it.plan_off), 1, M0all + it.m0_off,
                                       it.R0, it.R0, buf0, buf1, loc, outall ? outall + it.out_off : nullptr, L);
        __syncthreads();
        st_flush(L.s, sts + qi);
        __syncthreads();
    }
}

template <uint32_t FT>
static void launch_batch_t(gsi_ctx *c, uint32_t grid, const uint8_t *plans, const FBatchItem *items,
                           uint32_t nitems, const uint32_t *M0all, uint32_t *scratch, uint64_t slot_words,
                           uint32_t kmax, uint32_t *outall, FStatus *sts, uint32_t *counter, double bytes) {
    constexpr uint32_t CR = 4 * FT, CS = 16 * FT;
    launch(c, FT == 64 ? "k_fused_batch<64>" : FT == 256 ? "k_fused_batch<256>" : "k_fused_batch<1024>", bytes,
           k_fused_batch<FT, CR, CS>, grid, FT, plans, items, nitems, M0all, scratch, slot_words, kmax, outall, sts,
           counter);
}

// A few queries of a batch, each with nb workgroups of its own (at most one
// per CU over the launch).  The first workgroups of all of them come first in
// the grid, then every query's second one and so on.
__global__ __launch_bounds__(1024) void k_fused_cluster(const uint8_t *plans, const FClusterItem *items, uint32_t nitems,
                                                       uint32_t nb, uint64_t *ctl, uint32_t cl_rows, uint32_t cl_out,
                                                       ClusterWaits waits, FStatus *sts) {
    __shared__ FusedLds<1024, FUSED_MAX_ROWS, FUSED_MAX_SLOTS, true> L;
    __shared__ ClusterLds s_cl;
    const uint32_t i = blockIdx.x % nitems, bid = blockIdx.x / nitems;
    const FClusterItem it = items[i];
    st_clear(L.s);
    __syncthreads();
    Cluster cl{reinterpret_cast<ClusterCtl *>(ctl + (uint64_t)i * (CL_CTL_BYTES / 8)), bid, nb, 1u, cl_rows, cl_out, 0u, 0u,
               waits, &s_cl};
    fused_query<1024, FUSED_MAX_ROWS, FUSED_MAX_SLOTS, true, true>(reinterpret_cast<const FPlan *>(plans + it.plan_off),
                                                                   it.j0, it.M, it.R, it.R, it.buf0, it.buf1, it.loc,
                                                                   it.out, L, nullptr, 0, &cl);
    if (bid != 0) return;
    __syncthreads();
    st_flush(L.s, sts + i);
    if (nb > 1) cl_call(cl, 0, 0, 0, 0, 0);  // the helpers leave
}

void launch_fused_cluster(gsi_ctx *c, uint32_t nb, const uint8_t *plans, const FClusterItem *items, uint32_t nitems,
                          uint64_t *ctl, uint32_t cap_out, FStatus *sts) {
    launch(c, "k_fused_cluster", 0.0, k_fused_cluster, nb * nitems, 1024, plans, items, nitems, nb, ctl,
           cluster_table_rows(nb), cap_out, cluster_waits(c), sts);
}

// Chunks of one query (see launch_fused_chunks).  Every workgroup leaves
// once the chunk counter passes nchunks or the abort flag is set.
template <uint32_t FT, uint32_t CR, uint32_t CS>
__global__ __launch_bounds__(FT) void k_fused_chunks(const FPlan *plan, uint32_t j0, const uint32_t *M0, uint32_t R0,
                                                    uint32_t chunk_rows, uint32_t nchunks, uint32_t *scratch,
                                                    uint64_t slot_words, uint32_t k, uint32_t *staging,
                                                    uint64_t staging_words, unsigned long long *ocount,
                                                    uint32_t *abort, uint32_t max_fail, FStatus *sts,
                                                    uint32_t *counter, FChunkSummary *sum) {
    __shared__ FusedLds<FT, CR, CS, true> L;
    __shared__ uint32_t s_q;
    uint32_t *slot = scratch + (uint64_t)blockIdx.x * slot_words;
    uint32_t *buf0 = slot, *buf1 = slot + (uint64_t)CR * k, *loc = slot + 2ull * CR * k;
    // The only thread-0 block of the loop is at its head, and the chunk index
    // is made wave-uniform: the loop then stays one uniform loop around the
    // barriers (a thread-0 block after the last barrier let the compiler
    // split it so that the other lanes of wave 0 spun without thread 0).
    uint32_t prev = 0xFFFFFFFFu;  // chunk run last (read by thread 0 only)
    for (;;) {
        if (threadIdx.x == 0) {
            if (prev != 0xFFFFFFFFu) {
                // the chunk's status is still in LDS
                const FusedStat &p = L.s;
                if (p.head[ST_DONE]) {
                    // totals of the finished chunks
                    atomicAdd(&sum->digest[0], p.head[ST_DIG0]);
                    atomicXor(&sum->digest[1], p.head[ST_DIG1]);
                    atomicMax(&sum->levels, p.head[ST_LEVELS]);
                    for (uint32_t j = j0; j <= p.head[ST_LEVELS] && j < k; j++) {
                        atomicAdd(&sum->lv_rows[j], (uint64_t)p.lv[j]);
                        atomicAdd(&sum->lv_gba[j], (uint64_t)p.lv[GSI_MAX_K + j]);
                        atomicAdd(&sum->lv_surv[j], (uint64_t)p.lv[2 * GSI_MAX_K + j]);
                    }
                } else if (atomicAdd(abort + 1, 1u) + 1 > max_fail) {
                    // too many chunks that do not fit: leave the rest to the caller
                    atomicOr(abort, 1u);
                }
            }
            s_q = __atomic_load_n(abort, __ATOMIC_RELAXED) ? nchunks : atomicAdd(counter, 1u);
        }
        __syncthreads();
        const uint32_t qi = __builtin_amdgcn_readfirstlane(s_q);
        st_clear(L.s);
        __syncthreads();
        if (qi >= nchunks) break;
        const uint32_t first = qi * chunk_rows;
        const uint32_t rows = min(chunk_rows, R0 - first);
        fused_query<FT, CR, CS, true>(plan, j0, M0 + first, rows, R0, buf0, buf1, loc, staging, L, ocount,
                                      staging_words);
        prev = qi;
        __syncthreads();
        st_flush(L.s, sts + qi);
    }
}

// Each chunk's first output row (exclusive prefix of the counts, chunk
// order), its done flag, the row total and whether every chunk finished.
// The other totals were added by the chunk kernel.  One 1024-thread
// workgroup.
__global__ __launch_bounds__(1024) void k_chunk_summary(const FStatus *sts, uint32_t n, uint64_t *offs, uint32_t *done,
                                                       FChunkSummary *sum) {
    __shared__ uint64_t s_w[16];
    __shared__ uint32_t s_nd[16];
    const uint32_t tid = threadIdx.x, lane = lane_id(), w = tid >> 6;
    uint64_t carry = 0;
    uint32_t notdone = 0;
    for (uint32_t base = 0; base < n; base += 1024) {
        const uint32_t i = base + tid;
        uint64_t c = 0;
        if (i < n) {
            const bool d = sts[i].done != 0;
            c = d ? sts[i].count : 0ull;
            done[i] = d ? 1u : 0u;
            notdone += d ? 0u : 1u;
        }
        const uint64_t inc = wave_inclusive_sum(c);
        if (lane == 63) s_w[w] = inc;
        __syncthreads();
        uint64_t off = carry, tot = 0;
        for (uint32_t q = 0; q < 16; q++) {
            off += q < w ? s_w[q] : 0ull;
            tot += s_w[q];
        }
        if (i < n) offs[i] = off + inc - c;
        carry += tot;
        __syncthreads();
    }
    notdone = wave_sum(notdone);
    if (lane == 0) s_nd[w] = notdone;
    __syncthreads();
    if (tid == 0) {
        uint32_t nd = 0;
        for (uint32_t q = 0; q < 16; q++) nd += s_nd[q];
        offs[n] = carry;
        sum->all_done = nd == 0 ? 1u : 0u;
        sum->count = carry;
    }
}

// Rows of every finished chunk into `out`, in chunk order.  One workgroup
// per chunk.
__global__ __launch_bounds__(256) void k_chunk_gather(const FStatus *sts, const uint64_t *offs,
                                                     const uint32_t *staging, uint32_t k, uint32_t *out) {
    const FStatus &st = sts[blockIdx.x];
    if (!st.done) return;
    const uint64_t words = st.count * k;
    if (words == 0) return;
    const uint32_t *src = staging + st.out_base;
    uint32_t *dst = out + offs[blockIdx.x] * k;
    for (uint64_t t = threadIdx.x; t < words; t += 256) dst[t] = src[t];
}

template <uint32_t FT>
static void launch_chunks_t(gsi_ctx *c, uint32_t grid, const FPlan *plan, uint32_t j0, const uint32_t *M0, uint32_t R0,
                            uint32_t chunk_rows, uint32_t nchunks, uint32_t *scratch, uint64_t slot_words, uint32_t k,
                            uint32_t *staging, uint64_t staging_words, unsigned long long *ocount, uint32_t *abort,
                            uint32_t max_fail, FStatus *sts, uint32_t *counter, FChunkSummary *sum, double bytes) {
    constexpr uint32_t CR = 4 * FT, CS = 16 * FT;
    launch(c, "k_fused_chunks", bytes, k_fused_chunks<FT, CR, CS>, grid, FT, plan, j0, M0, R0, chunk_rows, nchunks,
           scratch, slot_words, k, staging, staging_words, ocount, abort, max_fail, sts, counter, sum);
}

void launch_fused_chunks(gsi_ctx *c, const FTier &t, uint32_t grid, const FPlan *plan, uint32_t j0, const uint32_t *M0,
                         uint32_t R0, uint32_t chunk_rows, uint32_t nchunks, uint32_t *scratch, uint64_t slot_words,
                         uint32_t k, uint32_t *staging, uint64_t staging_words, unsigned long long *ocount,
                         uint32_t *abort, uint32_t max_fail, FStatus *sts, uint32_t *counter, uint64_t *offs,
                         uint32_t *done, FChunkSummary *sum) {
    if (t.threads == 64)
        launch_chunks_t<64>(c, grid, plan, j0, M0, R0, chunk_rows, nchunks, scratch, slot_words, k, staging,
                            staging_words, ocount, abort, max_fail, sts, counter, sum, 0.0);
    else if (t.threads == 256)
        launch_chunks_t<256>(c, grid, plan, j0, M0, R0, chunk_rows, nchunks, scratch, slot_words, k, staging,
                             staging_words, ocount, abort, max_fail, sts, counter, sum, 0.0);
    else
        launch_chunks_t<1024>(c, grid, plan, j0, M0, R0, chunk_rows, nchunks, scratch, slot_words, k, staging,
                              staging_words, ocount, abort, max_fail, sts, counter, sum, 0.0);
    launch(c, "k_chunk_summary", 16.0 * nchunks, k_chunk_summary, 1, 1024, (const FStatus *)sts, nchunks, offs, done,
           sum);
}

void launch_chunk_gather(gsi_ctx *c, uint32_t nchunks, const FStatus *sts, const uint64_t *offs,
                         const uint32_t *staging, uint32_t k, uint32_t *out, uint64_t words) {
    launch(c, "k_chunk_gather", 8.0 * words, k_chunk_gather, nchunks, 256, sts, offs, staging, k, out);
}

// Rows of the given chunks, concatenated: workgroup i copies the `ncols`
// columns of chunk list[2i] to row list[2i+1] of dst (column stride `rows`).
__global__ __launch_bounds__(256) void k_take_rows(const uint32_t *M0, uint32_t R0, uint32_t ncols,
                                                  uint32_t chunk_rows, const uint32_t *list, uint32_t *dst,
                                                  uint64_t rows) {
    const uint32_t ch = list[2 * blockIdx.x], at = list[2 * blockIdx.x + 1];
    const uint32_t first = ch * chunk_rows;
    const uint32_t n = min(chunk_rows, R0 - first);
    for (uint32_t col = 0; col < ncols; col++)
        for (uint32_t t = threadIdx.x; t < n; t += 256)
            dst[(uint64_t)col * rows + at + t] = M0[(uint64_t)col * R0 + first + t];
}

void launch_take_rows(gsi_ctx *c, uint32_t nlist, const uint32_t *M0, uint32_t R0, uint32_t ncols,
                      uint32_t chunk_rows, const uint32_t *list, uint32_t *dst, uint64_t rows) {
    launch(c, "k_take_rows", 8.0 * rows * ncols, k_take_rows, nlist, 256, M0, R0, ncols, chunk_rows, list, dst,
           rows);
}

FTier fused_tier(uint32_t threads) {
    FTier t;
    t.threads = threads;
    t.cap_rows = 4 * threads;
    t.cap_slots = 16 * threads;
    int per_cu = 0;
    hipError_t e = hipSuccess;
    if (threads == 64)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_fused_batch<64, 256, 1024>, 64, 0);
    else if (threads == 256)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_fused_batch<256, 1024, 4096>, 256, 0);
    else
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_fused_batch<1024, 4096, 16384>, 1024, 0);
    if (e != hipSuccess || per_cu < 1) per_cu = 1;
    t.blocks_per_cu = (uint32_t)per_cu;
    return t;
}

void launch_fused_batch(gsi_ctx *c, const FTier &t, uint32_t grid, const uint8_t *plans, const FBatchItem *items,
                        uint32_t nitems, const uint32_t *M0all, uint32_t *scratch, uint64_t slot_words, uint32_t kmax,
                        uint32_t *outall, FStatus *sts, uint32_t *counter, double bytes) {
    if (t.threads == 64)
        launch_batch_t<64>(c, grid, plans, items, nitems, M0all, scratch, slot_words, kmax, outall, sts, counter, bytes);
    else if (t.threads == 256)
        launch_batch_t<256>(c, grid, plans, items, nitems, M0all, scratch, slot_words, kmax, outall, sts, counter,
                            bytes);
    else
        launch_batch_t<1024>(c, grid, plans, items, nitems, M0all, scratch, slot_words, kmax, outall, sts, counter,
                             bytes);
}

}  // namespace gsi
