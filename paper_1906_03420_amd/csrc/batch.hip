// The batched path: many queries over one resident graph.
//
//   filter   one pass of the signature filter per 32 query vertices of the
//            whole batch (query vertices grouped by label), one readback
//   plan     Algorithm 2 per query on the host
//   roots    every query's C(u_first) compacted in one pass
//   tier 1   persistent fused launch, workgroups of the scheduled size pull
//            queries from a shared counter and run all levels per query
//   tier 2   what tier 1 could not hold, in 1024-thread workgroups
//   clusters a few queries that are left then, several workgroups each
//   rest     the level-synchronous engine (wide.hip), all at once
//
// The schedule (tier-1 workgroup size, launched occupancy) is chosen by the
// autotuner, which times every candidate on a sample of the batch.
#include <algorithm>
#include <chrono>
#include <cstring>
#include <map>
#include <memory>

#include "admit.h"
#include "fused.h"
#include "gsi_internal.h"
#include "wide.h"

struct gsi_batch {
    gsi_ctx *ctx = nullptr;
    uint32_t nq = 0;
    bool count_only = false;
    std::unique_ptr<gsi::Slot[]> slots;
    gsi_batch_info info{};
};

namespace gsi {

constexpr uint32_t BQT = 256;
constexpr uint32_t TIER2_THREADS = 1024;

__global__ __launch_bounds__(BQT) void k_roots_popc(const uint64_t *bits, const uint32_t *rows, uint64_t nwords,
                                                   uint64_t total, uint32_t *cnt) {
    const uint64_t idx = (uint64_t)blockIdx.x * BQT + threadIdx.x;
    if (idx >= total) return;
    const uint64_t q = idx / nwords, wi = idx - q * nwords;
    cnt[idx] = (uint32_t)__popcll(bits[(uint64_t)rows[q] * nwords + wi]);
}

__global__ __launch_bounds__(BQT) void k_roots_emit(const uint64_t *bits, const uint32_t *rows, uint64_t nwords,
                                                   uint64_t total, const uint64_t *off, uint32_t *out) {
    const uint64_t idx = (uint64_t)blockIdx.x * BQT + threadIdx.x;
    if (idx >= total) return;
    const uint64_t q = idx / nwords, wi = idx - q * nwords;
    uint64_t b = bits[(uint64_t)rows[q] * nwords + wi];
    uint64_t o = off[idx];
    while (b) {
        const uint32_t t = (uint32_t)__ffsll((unsigned long long)b) - 1;
        out[o++] = (uint32_t)(wi * 64 + t);
        b &= b - 1;
    }
}

static uint32_t bgrid(uint64_t n) {
    uint64_t b = (n + BQT - 1) / BQT;
    if (b == 0) b = 1;
    if (b > 0x7FFFFFFFull) fail(GSI_E_CAPACITY, "grid too large");
    return (uint32_t)b;
}

static double ms_since(std::chrono::steady_clock::time_point t0) {
    return std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
}

static int cu_count(gsi_ctx *c) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, c->device) != hipSuccess || n < 1) n = 1;
    return n;
}

static void *round_block(gsi_ctx *c, uint64_t bytes, const char *what) {
    void *p = c->arena.alloc(bytes ? bytes : 256, false);
    if (!p)
        fail(GSI_E_NOMEM, "arena exhausted allocating %llu bytes for %s (largest free block %llu)",
             (unsigned long long)bytes, what, (unsigned long long)c->arena.largest_free());
    return p;
}

// An arena block with an owner.
struct TableBlock {
    gsi_ctx *c;
    void *p;
    TableBlock(gsi_ctx *ctx, uint64_t bytes, const char *what) : c(ctx), p(round_block(ctx, bytes, what)) {}
    TableBlock(const TableBlock &) = delete;
    TableBlock &operator=(const TableBlock &) = delete;
    ~TableBlock() {
        if (p) c->arena.release(p);
    }
};

struct FusedQuery {
    uint32_t qi;       // batch index
    uint32_t R0;
    uint64_t plan_off; // bytes
    uint64_t m0_off;   // rows
    uint64_t out_off;  // words
    // where it stands: level j of the table M (R rows x j columns)
    uint32_t j = 1;
    uint32_t *M = nullptr;
    uint32_t R = 0;
    std::shared_ptr<TableBlock> own;  // M's block, when it is not the root table
    uint32_t need = 2;  // workgroups it does not fit without, as far as its levels are known
};

// Workgroups without which a level that stopped a fused kernel does not fit:
// by its rows, its slots (sums over lists cut at what the kernel holds, so
// no more than the true ones) and, once joined, its survivors.
static uint32_t workgroups_needed(const FStatus &s, uint32_t k, bool count_only) {
    const uint64_t rows = s.rows, slots = s.lv_gba[s.level], surv = s.lv_surv[s.level];
    uint64_t n = std::max<uint64_t>(2, (rows + CL_CAP_ROWS / CL_MAX_WG - 1) / (CL_CAP_ROWS / CL_MAX_WG));
    n = std::max(n, (slots + CL_ROW_WEIGHT * rows + FUSED_MAX_SLOTS - 1) / FUSED_MAX_SLOTS);
    if (s.level + 1 < k) n = std::max(n, (surv + CL_CAP_ROWS / CL_MAX_WG - 1) / (CL_CAP_ROWS / CL_MAX_WG));
    else if (!count_only) n = std::max(n, (surv + CL_CAP_OUT / CL_MAX_WG - 1) / (CL_CAP_OUT / CL_MAX_WG));
    return (uint32_t)std::min<uint64_t>(n, 0xFFFFFFFFull);
}

// Runs one fused tier over `list`; fills entries of finished queries and
// returns the ones it could not hold.
static std::vector<FusedQuery> run_tier(gsi_graph *g, const std::shared_ptr<Round> &rd,
                                        const std::vector<Slot *> &slots, bool count_only, uint8_t path,
                                        const FTier &t,
                                        uint32_t grid_scale, const std::vector<FusedQuery> &list,
                                        const std::vector<uint32_t> &ks, const uint8_t *d_plans,
                                        const uint32_t *d_M0) {
    gsi_ctx *c = g->ctx;
    std::vector<FusedQuery> left;
    if (list.empty()) return left;
    const uint32_t n = (uint32_t)list.size();
    uint32_t kmax = 2;
    std::vector<FBatchItem> items(n);
    for (uint32_t i = 0; i < n; i++) {
        items[i].plan_off = list[i].plan_off;
        items[i].m0_off = list[i].m0_off;
        items[i].out_off = list[i].out_off;
        items[i].R0 = list[i].R0;
        kmax = std::max(kmax, ks[list[i].qi]);
    }
    const uint64_t per_cu = std::max<uint64_t>(1, (uint64_t)t.blocks_per_cu * grid_scale / 8);
    const uint32_t grid = (uint32_t)std::min<uint64_t>(n, per_cu * cu_count(c));
    const uint64_t slot_words = 2ull * t.cap_rows * kmax + fused_loc_words(kmax - 1, t.cap_rows);
    Scratch ts(c);
    FBatchItem *d_items = ts.get<FBatchItem>(n, "batch items");
    uint32_t *scratch = ts.get<uint32_t>(slot_words * grid, "batch slots");
    FStatus *d_st = reinterpret_cast<FStatus *>(ts.get<uint64_t>((uint64_t)n * sizeof(FStatus) / 8, "batch status"));
    uint32_t *counter = ts.get<uint32_t>(1, "batch counter");
    GSI_HIP(hipMemcpyAsync(d_items, items.data(), sizeof(FBatchItem) * n, hipMemcpyHostToDevice, c->stream));
    fill_u32(c, counter, 0, 1);
    launch_fused_batch(c, t, grid, d_plans, d_items, n, d_M0, scratch, slot_words, kmax, count_only ? nullptr : rd->out,
                       d_st, counter, 0.0);
    std::vector<FStatus> hs(n);
    GSI_HIP(hipMemcpyAsync(hs.data(), d_st, sizeof(FStatus) * n, hipMemcpyDeviceToHost, c->stream));
    sync(c);  // also keeps `items` alive until its copy has run
    for (uint32_t i = 0; i < n; i++) {
        Slot &sl = *slots[list[i].qi];
        if (hs[i].done) {
            sl.done = true;
            sl.path = path;
            sl.count = hs[i].count;
            sl.digest[0] = hs[i].digest[0];
            sl.digest[1] = hs[i].digest[1];
            if (!count_only && hs[i].count) {
                sl.rows = rd->out + list[i].out_off;
                sl.keep = rd;
            }
        } else {
            left.push_back(list[i]);
            left.back().need = workgroups_needed(hs[i], sl.k, count_only);
        }
    }
    return left;
}

// Runs each query of `list` with nb workgroups from where it stands, fills the
// entries of those that finish and returns the others, with the table each has
// reached (all of them as they were when the tables would take too much of the
// arena).
static std::vector<FusedQuery> run_clusters(gsi_graph *g, const std::vector<Slot *> &slots, bool count_only,
                                            uint32_t nb, const std::vector<FusedQuery> &list,
                                            const uint8_t *d_plans) {
    gsi_ctx *c = g->ctx;
    const uint32_t n = (uint32_t)list.size();
    const uint32_t rows = cluster_table_rows(nb), cap_out = cluster_result_rows(nb);
    uint64_t words = 0;
    for (auto &f : list) {
        const uint32_t k = slots[f.qi]->k;
        words += 2ull * rows * k + cluster_loc_words(k - 1, rows) + (count_only ? 0 : (uint64_t)cap_out * k);
    }
    if (4 * words > c->arena.largest_free() / 8) return list;
    std::vector<FClusterItem> items(n);
    std::vector<std::shared_ptr<TableBlock>> buf(2 * n);
    Scratch ts(c);
    for (uint32_t i = 0; i < n; i++) {
        Slot &sl = *slots[list[i].qi];
        if (!count_only) sl.own = persist<uint32_t>(c, (uint64_t)cap_out * sl.k, "cluster rows");
        for (uint32_t t = 0; t < 2; t++)
            buf[2 * i + t] = std::make_shared<TableBlock>(c, 4ull * rows * sl.k, "cluster tables");
        items[i].plan_off = list[i].plan_off;
        items[i].M = list[i].M;
        items[i].buf0 = static_cast<uint32_t *>(buf[2 * i]->p);
        items[i].buf1 = static_cast<uint32_t *>(buf[2 * i + 1]->p);
        items[i].loc = ts.get<uint32_t>(cluster_loc_words(sl.k - 1, rows), "cluster lookups");
        items[i].out = sl.own;
        items[i].R = list[i].R;
        items[i].j0 = list[i].j;
    }
    FClusterItem *d_items = ts.get<FClusterItem>(n, "cluster items");
    FStatus *d_st = reinterpret_cast<FStatus *>(ts.get<uint64_t>((uint64_t)n * sizeof(FStatus) / 8, "cluster status"));
    uint64_t *ctl = ts.get<uint64_t>(n * (CL_CTL_BYTES / 8), "cluster control");
    GSI_HIP(hipMemcpyAsync(d_items, items.data(), sizeof(FClusterItem) * n, hipMemcpyHostToDevice, c->stream));
    fill_u64(c, ctl, 0, n * (CL_CTL_BYTES / 8));
    launch_fused_cluster(c, nb, d_plans, d_items, n, ctl, cap_out, d_st);
    std::vector<FStatus> hs(n);
    GSI_HIP(hipMemcpyAsync(hs.data(), d_st, sizeof(FStatus) * n, hipMemcpyDeviceToHost, c->stream));
    sync(c);  // also keeps `items` alive until its copy has run
    std::vector<FusedQuery> left;
    for (uint32_t i = 0; i < n; i++) {
        Slot &sl = *slots[list[i].qi];
        if (hs[i].done) {
            sl.done = true;
            sl.path = PATH_TIER2;
            sl.count = hs[i].count;
            sl.digest[0] = hs[i].digest[0];
            sl.digest[1] = hs[i].digest[1];
        } else {
            left.push_back(list[i]);
            FusedQuery &f = left.back();
            f.need = workgroups_needed(hs[i], sl.k, count_only);
            if (hs[i].mloc != FSTATUS_IN_FIRST) {
                f.own = buf[2 * i + hs[i].mloc];
                f.M = static_cast<uint32_t *>(f.own->p);
                f.j = (uint32_t)hs[i].level;
                f.R = (uint32_t)hs[i].rows;
                c->arena.shrink(f.M, 4ull * f.R * f.j);
            }
        }
        if (!sl.own) continue;
        if (sl.done && sl.count) {
            c->arena.shrink(sl.own, sl.count * sl.k * 4);
            sl.rows = sl.own;
        } else {
            c->arena.release(sl.own);
            sl.own = nullptr;
        }
    }
    return left;
}

// A few queries that the tiers leave take several CUs each: in passes, each
// over as many of them as have the workgroups that their known levels need, at
// least half.  As soon as one is known to fit no number of workgroups, all that
// are left go on in the engine, whose steps take them along, from the tables
// they have reached; many go there at once.  Over 41 batches that leave 1 to
// 101 queries this is 1.30 times as fast as the engine alone (0.84 to 2.6), where
// passes to the end, starting over from the roots in the engine, were 1.06
// times (0.76 where one query was left in the end).  Sixteen queries of 10^6
// slots, four a pass, took 0.98 ms, in the engine 0.68.  (Before the 1024-thread
// tier, in its place: a batch of 131 small queries 0.57 -> 0.63 ms.)
static std::vector<FusedQuery> run_left(gsi_graph *g, const std::vector<Slot *> &slots, bool count_only,
                                        std::vector<FusedQuery> left, const uint8_t *d_plans) {
    for (uint32_t pass = 0; pass < CLB_PASSES && !left.empty() && left.size() <= CLB_MAX_QUERIES; pass++) {
        std::sort(left.begin(), left.end(), [](const FusedQuery &a, const FusedQuery &b) {
            return a.need != b.need ? a.need < b.need : a.qi < b.qi;
        });
        if (left.back().need > CL_MAX_WG) break;
        const uint32_t cus = (uint32_t)cu_count(g->ctx);
        size_t m = left.size();
        while (m && std::min<uint32_t>(CL_MAX_WG, cus / (uint32_t)m) < left[m - 1].need) m--;
        if (2 * m < left.size()) break;
        std::vector<FusedQuery> now(left.begin(), left.begin() + m);
        left.erase(left.begin(), left.begin() + m);
        now = run_clusters(g, slots, count_only, std::min<uint32_t>(CL_MAX_WG, cus / (uint32_t)m), now, d_plans);
        left.insert(left.end(), now.begin(), now.end());
    }
    return left;
}

void finish_slot(WideQuery &x, Slot &sl) {
    sl.done = true;
    sl.path = PATH_LEVELS;
    sl.status = x.status;
    sl.count = x.count;
    sl.digest[0] = x.digest[0];
    sl.digest[1] = x.digest[1];
    sl.own = x.take_rows();
    sl.rows = sl.own;
}

std::vector<WideQuery> admit_round(gsi_graph *g, const std::vector<const HostQuery *> &hq,
                                   const std::vector<Slot *> &slots, const std::vector<uint64_t> &tags,
                                   bool count_only, bool levels_only, gsi_batch_schedule sched, bool clusters,
                                   AdmitStats *st) {
    gsi_ctx *c = g->ctx;
    const uint32_t nq = (uint32_t)hq.size();
    std::vector<WideQuery> wide;
    auto rd = std::make_shared<Round>();
    rd->ctx = c;
    for (uint32_t i = 0; i < nq; i++) {
        slots[i]->ctx = c;
        slots[i]->k = hq[i]->k;
    }
    // queries whose edge labels G lacks have no match
    std::vector<uint32_t> active;
    for (uint32_t i = 0; i < nq; i++) {
        bool ok = true;
        for (uint32_t l : hq[i]->el) ok &= l < g->nlab && g->edges[l] > 0;
        if (ok) {
            active.push_back(i);
        } else {
            slots[i]->done = true;
            st->empty++;
        }
    }
    if (active.empty()) return wide;
    const uint64_t nwords = ((uint64_t)g->n + 63) / 64;
    std::vector<const HostQuery *> aq;
    std::vector<uint32_t> qbase{0};
    for (uint32_t i : active) {
        aq.push_back(hq[i]);
        qbase.push_back(qbase.back() + hq[i]->k);
    }
    const uint64_t nqv = qbase.back();
    auto tf = std::chrono::steady_clock::now();
    rd->bits = round_block(c, nqv * nwords * 8, "candidate bitsets");
    uint64_t *bits = static_cast<uint64_t *>(rd->bits);
    std::vector<uint32_t> cnt(nqv);
    {
        Scratch fs(c);
        uint32_t *dcnt = fs.get<uint32_t>(nqv, "candidate counts");
        run_filter_many(g, aq, qbase, bits, dcnt);
        GSI_HIP(hipMemcpyAsync(cnt.data(), dcnt, 4 * nqv, hipMemcpyDeviceToHost, c->stream));
        sync(c);
    }
    st->filter_ms += std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - tf).count();

    const FTier t1 = fused_tier(sched.threads), t2 = fused_tier(TIER2_THREADS);
    std::vector<uint32_t> ks(nq);
    for (uint32_t i = 0; i < nq; i++) ks[i] = hq[i]->k;
    struct Planned {
        uint32_t qi, a;
        std::vector<uint32_t> order, e0src;
        std::vector<uint32_t> cand;
        uint32_t R0;
        uint64_t m0_off;
    };
    std::vector<Planned> planned;
    std::vector<uint32_t> single;
    for (size_t a = 0; a < active.size(); a++) {
        const uint32_t qi = active[a];
        const HostQuery &q = *hq[qi];
        std::vector<uint32_t> cand(cnt.begin() + qbase[a], cnt.begin() + qbase[a] + q.k);
        bool empty = false;
        for (uint32_t x : cand) empty |= x == 0;
        if (empty) {
            slots[qi]->done = true;
            st->empty++;
            continue;
        }
        if (q.k < 2) {
            single.push_back(qi);
            continue;
        }
        Planned pl;
        pl.qi = qi;
        pl.a = (uint32_t)a;
        make_plan(g, q, cand, pl.order, pl.e0src);
        pl.R0 = cand[pl.order[0]];
        pl.m0_off = 0;
        pl.cand = cand;
        planned.push_back(std::move(pl));
    }

    const uint32_t max_roots = clusters ? CL_TAKE_ROWS : t2.cap_rows;
    std::vector<FusedQuery> fused;
    std::vector<uint8_t> plan_blob;
    std::vector<uint32_t> root_rows;
    uint64_t m0_total = 0, out_total = 0;
    for (auto &pl : planned) {
        const HostQuery &q = *hq[pl.qi];
        pl.m0_off = m0_total;
        m0_total += pl.R0;
        root_rows.push_back(qbase[pl.a] + pl.order[0]);
        if (levels_only || pl.R0 > max_roots) continue;
        uint32_t n_edges = 0;
        for (uint32_t j = 1; j < q.k; j++)
            for (uint32_t i = 0; i < j; i++)
                for (auto &p : q.adj[pl.order[j]]) n_edges += p.first == pl.order[i];
        const size_t pb = (fplan_bytes(n_edges) + 15) & ~size_t(15);
        const uint64_t off = plan_blob.size();
        plan_blob.resize(off + pb, 0);
        FPlan *hp = reinterpret_cast<FPlan *>(plan_blob.data() + off);
        hp->k = q.k;
        hp->count_only = count_only ? 1u : 0u;
        hp->cap_rows = 0xFFFFFFFFu;  // the tier's own capacities apply
        hp->cap_slots = 0xFFFFFFFFu;
        hp->pick = 1;
        hp->ci_all = g->ci;
        std::vector<uint32_t> col(q.k);
        for (uint32_t j = 0; j < q.k; j++) col[pl.order[j]] = j;
        for (uint32_t v = 0; v < q.k; v++) hp->qcol[v] = col[v];
        uint32_t ei = 0;
        for (uint32_t j = 1; j < q.k; j++) {
            hp->lv_first[j] = ei;
            hp->Cu[j] = bits + (uint64_t)(qbase[pl.a] + pl.order[j]) * nwords;
            uint32_t ne = 0;
            for (uint32_t i = 0; i < j; i++)
                for (auto &p : q.adj[pl.order[j]])
                    if (p.first == pl.order[i]) {
                        const uint32_t l = p.second;
                        FEdge &fe = hp->edges[ei + ne];
                        fe.gl = g->gl + g->group_base[l] * GROUP_WORDS;
                        fe.ci = g->ci + g->ci_base[l];
                        fe.G = g->G[l];
                        fe.H = g->H[l];
                        fe.col = i;
                        fe.ci_off = (uint32_t)g->ci_base[l];
                        if (pl.order[i] == pl.e0src[j]) hp->lv_e0[j] = ne;
                        ne++;
                    }
            hp->lv_ne[j] = ne;
            hp->lv_mmask[j] = 0;
            for (uint32_t c = 0; c < j; c++)
                if (q.multi || q.vl[pl.order[c]] == q.vl[pl.order[j]]) hp->lv_mmask[j] |= 1u << c;
            ei += ne;
        }
        FusedQuery f;
        f.qi = pl.qi;
        f.R0 = pl.R0;
        f.plan_off = off;
        f.m0_off = pl.m0_off;
        f.out_off = out_total;
        if (pl.R0 <= t2.cap_rows) out_total += count_only ? 0 : (uint64_t)t2.cap_slots * q.k;
        fused.push_back(f);
    }

    std::vector<uint32_t> to_wide;
    std::map<uint32_t, FusedQuery> stand;  // those of them that a fused kernel has seen
    uint32_t *d_M0 = nullptr;
    if (!planned.empty()) {
        Scratch rs(c);
        uint32_t *d_rows = rs.get<uint32_t>(root_rows.size(), "root rows");
        GSI_HIP(hipMemcpyAsync(d_rows, root_rows.data(), 4 * root_rows.size(), hipMemcpyHostToDevice, c->stream));
        const uint64_t tw = (uint64_t)root_rows.size() * nwords;
        rd->m0 = round_block(c, m0_total * 4, "root tables");
        d_M0 = static_cast<uint32_t *>(rd->m0);
        uint32_t *wc = rs.get<uint32_t>(tw, "root word counts");
        uint64_t *wo = rs.get<uint64_t>(tw + 1, "root word offsets");
        launch(c, "k_roots_popc", 12.0 * tw, k_roots_popc, bgrid(tw), BQT, (const uint64_t *)bits,
               (const uint32_t *)d_rows, nwords, tw, wc);
        exclusive_scan(c, wc, tw, wo, rs);
        launch(c, "k_roots_emit", 16.0 * tw + 4.0 * m0_total, k_roots_emit, bgrid(tw), BQT, (const uint64_t *)bits,
               (const uint32_t *)d_rows, nwords, tw, (const uint64_t *)wo, d_M0);
        sync(c);  // host vectors copied above stay alive until here
    }
    if (!fused.empty()) {
        for (auto &f : fused) {
            f.M = d_M0 + f.m0_off;
            f.R = f.R0;
        }
        Scratch ps(c);
        uint8_t *d_plans = ps.get<uint8_t>(plan_blob.size(), "fused plans");
        GSI_HIP(hipMemcpyAsync(d_plans, plan_blob.data(), plan_blob.size(), hipMemcpyHostToDevice, c->stream));
        if (!count_only && out_total) rd->out = static_cast<uint32_t *>(round_block(c, out_total * 4, "fused rows"));
        std::vector<FusedQuery> first, second, large;
        for (auto &f : fused) (f.R0 <= t1.cap_rows ? first : f.R0 <= t2.cap_rows ? second : large).push_back(f);
        auto ta = std::chrono::steady_clock::now();
        std::vector<FusedQuery> left = run_tier(g, rd, slots, count_only, PATH_TIER1, t1, sched.grid_scale, first, ks, d_plans, d_M0);
        st->tier1 += (uint32_t)(first.size() - left.size());
        st->tier1_ms += std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - ta).count();
        second.insert(second.end(), left.begin(), left.end());
        auto tb = std::chrono::steady_clock::now();
        std::vector<FusedQuery> left2 = second;
        if (t1.threads != t2.threads)
            left2 = run_tier(g, rd, slots, count_only, PATH_TIER2, t2, 8, second, ks, d_plans, d_M0);
        for (auto &f : large) f.need = (f.R0 + CL_CAP_ROWS / CL_MAX_WG - 1) / (CL_CAP_ROWS / CL_MAX_WG);
        left2.insert(left2.end(), large.begin(), large.end());
        if (clusters) left2 = run_left(g, slots, count_only, std::move(left2), d_plans);
        st->tier2 += (uint32_t)(second.size() + large.size() - left2.size());
        st->tier2_ms += std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - tb).count();
        for (auto &f : left2) {
            to_wide.push_back(f.qi);
            stand.emplace(f.qi, std::move(f));
        }
    }
    for (auto &pl : planned)
        if (levels_only || pl.R0 > max_roots) to_wide.push_back(pl.qi);

    // one-vertex queries: the root table is the answer
    for (uint32_t qi : single) {
        gsi_query_options o{};
        o.flags = count_only ? GSI_COUNT_ONLY : 0u;
        gsi_result *r = run_query(g, *hq[qi], &o);
        Slot &sl = *slots[qi];
        sl.res = r;
        sl.done = true;
        sl.path = PATH_SINGLE;
        sl.count = r->count;
        sl.digest[0] = r->digest[0];
        sl.digest[1] = r->digest[1];
        sl.rows = r->rows;
        st->single++;
    }

    std::sort(to_wide.begin(), to_wide.end());
    std::vector<const Planned *> byq(nq, nullptr);
    for (auto &pl : planned) byq[pl.qi] = &pl;
    for (uint32_t qi : to_wide) {
        const Planned &pl = *byq[qi];
        const HostQuery &q = *hq[qi];
        WideQuery x;
        x.ctx = c;
        x.q = &q;
        x.qi = qi;
        x.tag = tags.empty() ? qi : tags[qi];
        x.keep = rd;
        x.order = pl.order;
        x.e0src = pl.e0src;
        x.cand = pl.cand;
        x.col.assign(q.k, 0);
        for (uint32_t j = 0; j < q.k; j++) x.col[pl.order[j]] = j;
        x.Cu.assign(q.k, nullptr);
        for (uint32_t j = 0; j < q.k; j++) x.Cu[j] = bits + (uint64_t)(qbase[pl.a] + pl.order[j]) * nwords;
        x.root = x.M = d_M0 + pl.m0_off;
        x.root_rows = x.R = pl.R0;
        const auto at = stand.find(qi);
        if (at != stand.end() && at->second.own) {
            // from the table a cluster has reached
            FusedQuery &f = at->second;
            x.j = f.j;
            x.M = f.M;
            x.R = f.R;
            x.own = f.own->p;
            f.own->p = nullptr;
        }
        wide.push_back(std::move(x));
    }
    st->wide += (uint32_t)wide.size();
    return wide;
}

gsi_batch *run_batch(gsi_graph *g, uint32_t nq, const gsi_query_desc *qd, uint32_t flags,
                     gsi_batch_schedule sched) {
    gsi_ctx *c = g->ctx;
    auto t0 = std::chrono::steady_clock::now();
    if (flags & ~(GSI_COUNT_ONLY | GSI_BATCH_LEVELS_ONLY)) fail(GSI_E_INVALID, "unknown batch flag");
    if (sched.threads != 64 && sched.threads != 256 && sched.threads != 1024)
        fail(GSI_E_INVALID, "schedule threads must be 64, 256 or 1024");
    if (sched.grid_scale < 1 || sched.grid_scale > 8) fail(GSI_E_INVALID, "schedule grid_scale must be 1..8");
    if (sched.engine_tiles > 8 || (sched.engine_tiles & (sched.engine_tiles - 1)))
        fail(GSI_E_INVALID, "schedule engine_tiles must be 0, 1, 2, 4 or 8");
    std::vector<HostQuery> hq(nq);
    for (uint32_t i = 0; i < nq; i++) {
        try {
            hq[i] = validate_query(qd[i].k, qd[i].vertex_labels, qd[i].n_edges, qd[i].src, qd[i].dst,
                                   qd[i].edge_labels);
        } catch (const Fail &f) {
            std::string m = std::string("query ") + std::to_string(i) + ": " + gsi_last_error();
            fail(f.st, "%s", m.c_str());
        }
    }
    std::unique_ptr<gsi_batch> b(new gsi_batch());
    b->ctx = c;
    b->nq = nq;
    b->count_only = (flags & GSI_COUNT_ONLY) != 0;
    b->slots.reset(new Slot[nq]);
    b->info.queries = nq;
    b->info.schedule = sched;
    std::vector<const HostQuery *> hp(nq);
    std::vector<Slot *> sp(nq);
    for (uint32_t i = 0; i < nq; i++) {
        hp[i] = &hq[i];
        sp[i] = &b->slots[i];
    }
    AdmitStats as;
    std::vector<WideQuery> wq = admit_round(g, hp, sp, {}, b->count_only, (flags & GSI_BATCH_LEVELS_ONLY) != 0,
                                            sched, true, &as);
    auto tw0 = std::chrono::steady_clock::now();
    wide_run(g, wq, b->count_only, sched.engine_tiles);
    for (auto &x : wq) finish_slot(x, b->slots[x.qi]);
    b->info.empty = as.empty;
    b->info.tier1 = as.tier1;
    b->info.tier2 = as.tier2;
    b->info.per_level = as.wide + as.single;
    b->info.filter_ms = as.filter_ms;
    b->info.tier1_ms = as.tier1_ms;
    b->info.tier2_ms = as.tier2_ms;
    b->info.per_level_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - tw0).count();
    b->info.total_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    return b.release();
}

}  // namespace gsi

using namespace gsi;

namespace {
const Slot &entry(const gsi_batch *b, uint32_t qi) {
    if (!b) fail(GSI_E_INVALID, "null batch");
    if (qi >= b->nq) fail(GSI_E_INVALID, "query index %u out of range (batch of %u)", qi, b->nq);
    return b->slots[qi];
}
}  // namespace

extern "C" {

gsi_status gsi_batch_run(gsi_graph *g, uint32_t nq, const gsi_query_desc *qs, const gsi_batch_options *opt,
                         gsi_batch **out) {
    GSI_TRY({
        if (!g || !out || (nq && !qs)) fail(GSI_E_INVALID, "null argument");
        if (g->multi) fail(GSI_E_INVALID, "multi-labelled graphs run through gsi_query_run_multi only");
        *out = nullptr;
        gsi_batch_schedule sc = opt ? opt->schedule : gsi_batch_schedule{0, 0};
        if (sc.threads == 0) sc = g->tuned;
        if (sc.threads == 0) sc = gsi_batch_schedule{256, 8, 0};
        gsi_ctx *c = g->ctx;
        Busy busy(c);
        GSI_HIP(hipSetDevice(c->device));
        *out = run_batch(g, nq, qs, opt ? opt->flags : 0u, sc);
    })
}

gsi_status gsi_batch_count(const gsi_batch *b, uint32_t qi, uint64_t *rows) {
    GSI_TRY({
        const auto &e = entry(b, qi);
        if (!rows) fail(GSI_E_INVALID, "null argument");
        *rows = e.count;
    })
}

gsi_status gsi_batch_digest(const gsi_batch *b, uint32_t qi, uint64_t out[2]) {
    GSI_TRY({
        const auto &e = entry(b, qi);
        if (!out) fail(GSI_E_INVALID, "null argument");
        out[0] = e.digest[0];
        out[1] = e.digest[1];
    })
}

gsi_status gsi_batch_results(const gsi_batch *b, uint64_t *counts, uint64_t *digests) {
    GSI_TRY({
        if (!b || !counts || !digests) fail(GSI_E_INVALID, "null argument");
        for (uint32_t qi = 0; qi < b->nq; qi++) {
            counts[qi] = b->slots[qi].count;
            digests[2 * (uint64_t)qi] = b->slots[qi].digest[0];
            digests[2 * (uint64_t)qi + 1] = b->slots[qi].digest[1];
        }
    })
}

gsi_status gsi_batch_rows(const gsi_batch *b, uint32_t qi, uint32_t *dst, uint64_t cap) {
    GSI_TRY({
        const auto &e = entry(b, qi);
        if (b->count_only) fail(GSI_E_INVALID, "batch was run with GSI_COUNT_ONLY");
        if (cap < e.count) fail(GSI_E_CAPACITY, "need %llu rows", (unsigned long long)e.count);
        if (e.count == 0) return GSI_OK;
        if (!dst) fail(GSI_E_INVALID, "null buffer");
        gsi_ctx *c = b->ctx;
        GSI_HIP(hipSetDevice(c->device));
        GSI_HIP(hipMemcpyAsync(dst, e.rows, e.count * e.k * 4, hipMemcpyDeviceToHost, c->stream));
        GSI_HIP(hipStreamSynchronize(c->stream));
    })
}

gsi_status gsi_batch_get_info(const gsi_batch *b, gsi_batch_info *out) {
    GSI_TRY({
        if (!b || !out) fail(GSI_E_INVALID, "null argument");
        *out = b->info;
    })
}

gsi_status gsi_batch_free(gsi_batch *b) {
    GSI_TRY({
        if (!b) return GSI_OK;
        gsi_ctx *c = b->ctx;
        GSI_HIP(hipSetDevice(c->device));
        GSI_HIP(hipStreamSynchronize(c->stream));
        delete b;
    })
}

gsi_status gsi_batch_tune(gsi_graph *g, uint32_t nq, const gsi_query_desc *qs, uint32_t sample,
                          gsi_batch_schedule *out, double *out_ms) {
    GSI_TRY({
        if (!g || !out || (nq && !qs)) fail(GSI_E_INVALID, "null argument");
        if (g->multi) fail(GSI_E_INVALID, "multi-labelled graphs run through gsi_query_run_multi only");
        gsi_ctx *c = g->ctx;
        Busy busy(c);
        GSI_HIP(hipSetDevice(c->device));
        const uint32_t n = std::max<uint32_t>(1, std::min(nq, sample ? sample : 128u));
        if (nq == 0) fail(GSI_E_INVALID, "no queries to tune on");
        const gsi_batch_schedule cands[] = {{64, 8, 0},  {64, 4, 0},   {256, 8, 0},
                                            {256, 4, 0}, {1024, 8, 0}, {1024, 4, 0}};
        double best = 1e300;
        gsi_batch_schedule win{256, 8, 0};
        auto trial = [&](const gsi_batch_schedule &sc) {
            auto t0 = std::chrono::steady_clock::now();
            gsi_batch *b = run_batch(g, n, qs, GSI_COUNT_ONLY, sc);
            double ms = ms_since(t0);
            delete b;
            if (ms < best) {
                best = ms;
                win = sc;
            }
        };
        for (const auto &sc : cands) trial(sc);
        // the engine's tiles per workgroup, with the fused tiers chosen
        const gsi_batch_schedule tiers = win;
        for (uint32_t tiles : {1u, 2u, 8u}) trial(gsi_batch_schedule{tiers.threads, tiers.grid_scale, tiles});
        if (win.engine_tiles == 0) win.engine_tiles = 4;
        g->tuned = win;
        *out = win;
        if (out_ms) *out_ms = best / n;
    })
}

}  // extern "C"
