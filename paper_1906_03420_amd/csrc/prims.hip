// Data-parallel primitives: fill, exclusive scan (u32 -> u64) and stable LSD
// radix sorts of 64-bit keys and of triples of uint32.  wave64 throughout.
#include "gsi_internal.h"

namespace gsi {

// ------------------------------------------------------------------- fill
template <typename T>
__global__ void k_fill(T *p, T v, uint64_t n) {
    uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = v;
}

static uint32_t grid_for(uint64_t n, uint32_t per_block, uint32_t cap = 65536) {
    uint64_t b = (n + per_block - 1) / per_block;
    if (b == 0) b = 1;
    if (b > cap) b = cap;
    return (uint32_t)b;
}

void fill_u32(gsi_ctx *c, uint32_t *p, uint32_t v, uint64_t n) {
    if (!n) return;
    launch(c, "k_fill", 4.0 * n, k_fill<uint32_t>, grid_for(n, 1024), 256, p, v, n);
}
void fill_u64(gsi_ctx *c, uint64_t *p, uint64_t v, uint64_t n) {
    if (!n) return;
    launch(c, "k_fill", 8.0 * n, k_fill<uint64_t>, grid_for(n, 1024), 256, p, v, n);
}

// ------------------------------------------------------------------- scan
// Three passes: per-tile sums, one-workgroup scan of the tile sums, and a
// per-tile scan that adds the tile's offset.  A tile is 256 threads x 8
// consecutive items.
constexpr int SCAN_THREADS = 256;
constexpr int SCAN_ITEMS = 8;
constexpr int SCAN_TILE = SCAN_THREADS * SCAN_ITEMS;

template <int NT>
__device__ uint64_t block_exclusive_sum(uint64_t v, uint64_t *total) {
    __shared__ uint64_t s_w[NT / 64];
    uint64_t inc = wave_inclusive_sum(v);
    const uint32_t lane = lane_id(), w = threadIdx.x >> 6;
    if (lane == 63) s_w[w] = inc;
    __syncthreads();
    uint64_t off = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < NT / 64; i++) {
        uint64_t x = s_w[i];
        off += (i < (int)w) ? x : 0;
        tot += x;
    }
    __syncthreads();
    *total = tot;
    return off + inc - v;
}

__global__ __launch_bounds__(SCAN_THREADS) void k_scan_reduce(const uint32_t *in, uint64_t n, uint64_t *part) {
    uint64_t base = (uint64_t)blockIdx.x * SCAN_TILE;
    uint64_t s = 0;
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; i++) {
        uint64_t idx = base + (uint64_t)i * SCAN_THREADS + threadIdx.x;
        if (idx < n) s += in[idx];
    }
    uint64_t tot;
    block_exclusive_sum<SCAN_THREADS>(s, &tot);
    if (threadIdx.x == 0) part[blockIdx.x] = tot;
}

__global__ __launch_bounds__(1024) void k_scan_partials(uint64_t *part, uint64_t nb, uint64_t *total,
                                                       uint64_t *total2, uint64_t *seqp, uint64_t seqv) {
    uint64_t carry = 0;
    for (uint64_t c0 = 0; c0 < nb; c0 += 1024) {
        uint64_t idx = c0 + threadIdx.x;
        uint64_t v = idx < nb ? part[idx] : 0;
        uint64_t tot;
        uint64_t ex = block_exclusive_sum<1024>(v, &tot);
        if (idx < nb) part[idx] = carry + ex;
        carry += tot;
    }
    if (threadIdx.x == 0) {
        *total = carry;
        if (total2) *total2 = carry;
        post_seq(seqp, seqv);
    }
}

__global__ __launch_bounds__(SCAN_THREADS) void k_scan_apply(const uint32_t *in, uint64_t n, const uint64_t *part,
                                                             uint64_t *out) {
    uint64_t base = (uint64_t)blockIdx.x * SCAN_TILE + (uint64_t)threadIdx.x * SCAN_ITEMS;
    uint32_t v[SCAN_ITEMS];
    uint64_t s = 0;
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; i++) {
        uint64_t idx = base + i;
        v[i] = idx < n ? in[idx] : 0;
        s += v[i];
    }
    uint64_t tot;
    uint64_t run = part[blockIdx.x] + block_exclusive_sum<SCAN_THREADS>(s, &tot);
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; i++) {
        uint64_t idx = base + i;
        if (idx < n) out[idx] = run;
        run += v[i];
    }
}

// whole scan in one workgroup, rounds of 1024 threads x 8 consecutive items:
// one launch instead of three.  A round's sums go through LDS, so that they
// are written in order.  With `slots` the items are the tiles of *slots slots
// (`per` each), none when there are more than `cap`.
__global__ __launch_bounds__(1024) void k_scan_small(const uint32_t *in, uint64_t n, uint64_t *out, uint64_t *total,
                                                    uint64_t *seqp, uint64_t seqv, const uint64_t *slots,
                                                    uint32_t per, uint64_t cap) {
    constexpr uint32_t ROUND = 1024 * SCAN_ITEMS;
    __shared__ uint64_t s_out[ROUND + ROUND / 16];  // one spare word in 16: a thread's 8 words start at 16 banks
    if (slots) {
        const uint64_t g = *slots;
        n = g > cap ? 0 : (g + per - 1) / per;
    }
    uint64_t carry = 0;
    for (uint64_t c0 = 0; c0 < n; c0 += ROUND) {
        const uint64_t base = c0 + (uint64_t)threadIdx.x * SCAN_ITEMS;
        uint32_t v[SCAN_ITEMS];
        uint64_t s = 0;
        if (base + SCAN_ITEMS <= n) {
            const uint4 *q = reinterpret_cast<const uint4 *>(in + base);  // `in` is 16-byte aligned
#pragma unroll
            for (int i = 0; i < SCAN_ITEMS / 4; i++) {
                const uint4 x = q[i];
                v[4 * i] = x.x;
                v[4 * i + 1] = x.y;
                v[4 * i + 2] = x.z;
                v[4 * i + 3] = x.w;
            }
        } else {
#pragma unroll
            for (int i = 0; i < SCAN_ITEMS; i++) v[i] = base + i < n ? in[base + i] : 0;
        }
#pragma unroll
        for (int i = 0; i < SCAN_ITEMS; i++) s += v[i];
        uint64_t tot;
        uint64_t run = carry + block_exclusive_sum<1024>(s, &tot);
#pragma unroll
        for (int i = 0; i < SCAN_ITEMS; i++) {
            const uint32_t x = threadIdx.x * SCAN_ITEMS + i;
            s_out[x + x / 16] = run;
            run += v[i];
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < SCAN_ITEMS; i++) {
            const uint32_t x = i * 1024 + threadIdx.x;
            if (c0 + x < n) out[c0 + x] = s_out[x + x / 16];
        }
        carry += tot;
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        out[n] = carry;
        if (total) *total = carry;
        post_seq(seqp, seqv);
    }
}

// items up to which one workgroup scans, in rounds of 8,192
constexpr uint64_t SMALL_SCAN = 4 * 8192;

void exclusive_scan(gsi_ctx *c, const uint32_t *in, uint64_t n, uint64_t *out, Scratch &s, uint64_t *total) {
    if (n == 0) {
        fill_u64(c, out, 0, 1);
        if (total) fill_u64(c, total, 0, 1);
        return;
    }
    uint64_t seqv = 0;
    uint64_t *seqp = seq_slot(c, total, &seqv);
    if (n <= SMALL_SCAN && (reinterpret_cast<uintptr_t>(in) & 15) == 0) {
        launch(c, "k_scan_small", 12.0 * n, k_scan_small, 1, 1024, in, n, out, total, seqp, seqv,
               (const uint64_t *)nullptr, 0u, (uint64_t)0);
        c->seq_armed = seqp != nullptr;
        return;
    }
    uint64_t nb = (n + SCAN_TILE - 1) / SCAN_TILE;
    if (nb > 0x7FFFFFFFull) fail(GSI_E_INVALID, "scan too large");
    uint64_t *part = s.get<uint64_t>(nb, "scan partials");
    launch(c, "k_scan_reduce", 4.0 * n, k_scan_reduce, (uint32_t)nb, SCAN_THREADS, in, n, part);
    launch(c, "k_scan_partials", 16.0 * nb, k_scan_partials, 1, 1024, part, nb, out + n, total, seqp, seqv);
    launch(c, "k_scan_apply", 12.0 * n, k_scan_apply, (uint32_t)nb, SCAN_THREADS, in, n, (const uint64_t *)part, out);
    // the total is posted before the apply pass ends; a reader of it alone
    // need not wait for out[]: stream order makes later launches see out[]
    c->seq_armed = seqp != nullptr;
    s.drop(part);
}

void exclusive_scan_tiles(gsi_ctx *c, const uint32_t *in, const uint64_t *slots, uint32_t per, uint64_t cap,
                          uint64_t *out, uint64_t *total) {
    uint64_t seqv = 0;
    uint64_t *seqp = seq_slot(c, total, &seqv);
    const double tiles = (double)((cap + per - 1) / per);
    launch(c, "k_scan_small", 12.0 * tiles, k_scan_small, 1, 1024, in, (uint64_t)0, out, total, seqp, seqv, slots,
           per, cap);
    c->seq_armed = seqp != nullptr;
}

// ------------------------------------------------------- 64-bit key sort
// Stable LSD radix sort of 64-bit keys, up to 8 bits a pass: a histogram of
// every tile, one launch that turns them into each tile's first place per
// digit, and a scatter.  The scatter orders its tile by digit in LDS first,
// so that it writes runs of keys (on average tile / 256 of them) instead of
// one key per lane and place, and a wave ranks its keys against counters of
// its own, so that the rounds need no barrier.  A pass is bound by HBM: 24
// bytes a key with the histogram.  Over 2*10^8 entries three 32-bit arrays
// scattered from registers took 3.8 ms a scatter (1.3 TB/s); the packed keys
// take 0.7 ms (4.6 TB/s), a histogram 0.3 ms.
struct KeyArray {
    const uint64_t *k;
    __device__ __forceinline__ uint64_t operator()(uint32_t p) const { return k[p]; }
};
// entry p of the directed edges: edge p / 2 from its source (even p) or its
// destination, packed as label, source, destination (vb bits an end)
struct EdgeKeys {
    const uint32_t *src, *dst, *el;
    int vb;
    __device__ __forceinline__ uint64_t operator()(uint32_t p) const {
        const uint32_t e = p >> 1;
        const uint32_t a = src[e], b = dst[e], l = el[e];
        const uint32_t s = (p & 1) ? b : a, d = (p & 1) ? a : b;
        return ((uint64_t)l << (2 * vb)) | ((uint64_t)s << vb) | d;
    }
};

constexpr uint32_t KS_BINS = 256;

// lanes of this wave holding the same digit of `bits` bits (valid lanes only)
__device__ __forceinline__ uint64_t digit_peers(uint32_t d, int bits, bool valid) {
    uint64_t peers = __ballot(valid);
    for (int b = 0; b < bits; b++) {
        const bool bit = (d >> b) & 1u;
        const uint64_t bb = __ballot(valid && bit);
        peers &= bit ? bb : ~bb;
    }
    return valid ? peers : 0ull;
}

template <uint32_t NT, uint32_t ITEMS, typename In>
__global__ __launch_bounds__(NT) void k_key_hist(In in, int shift, int bits, uint32_t n, uint32_t ntiles,
                                                 uint32_t *hist) {
    // a copy per wave: equal digits of different waves do not meet
    __shared__ uint32_t h[NT / 64][KS_BINS];
    const uint32_t t = threadIdx.x, w = t >> 6, mask = (1u << bits) - 1;
    for (uint32_t i = t; i < NT / 64 * KS_BINS; i += NT) (&h[0][0])[i] = 0;
    __syncthreads();
    const uint64_t base = (uint64_t)blockIdx.x * (NT * ITEMS);
    uint32_t d[ITEMS];
#pragma unroll
    for (uint32_t r = 0; r < ITEMS; r++) {
        const uint64_t p = base + r * NT + t;
        d[r] = (uint32_t)(in((uint32_t)(p < n ? p : n - 1)) >> shift) & mask;
    }
#pragma unroll
    for (uint32_t r = 0; r < ITEMS; r++)
        if (base + r * NT + t < n) atomicAdd(&h[w][d[r]], 1u);
    __syncthreads();
    for (uint32_t b = t; b <= mask; b += NT) {
        uint32_t sum = 0;
#pragma unroll
        for (uint32_t q = 0; q < NT / 64; q++) sum += h[q][b];
        hist[(uint64_t)b * ntiles + blockIdx.x] = sum;
    }
}

// hist row b (ntiles counts) -> exclusive prefix sums in place, tot[b] = sum;
// one workgroup per digit, 8 consecutive counts a thread
__global__ __launch_bounds__(1024) void k_key_offsets(uint32_t *hist, uint32_t ntiles, uint32_t *tot) {
    uint32_t *row = hist + (uint64_t)blockIdx.x * ntiles;
    uint32_t carry = 0;
    for (uint32_t c0 = 0; c0 < ntiles; c0 += 8192) {
        uint32_t v[8];
        uint64_t sum = 0;
#pragma unroll
        for (uint32_t i = 0; i < 8; i++) {
            const uint32_t x = c0 + threadIdx.x * 8 + i;
            v[i] = x < ntiles ? row[x] : 0u;
            sum += v[i];
        }
        uint64_t all;
        uint32_t run = carry + (uint32_t)block_exclusive_sum<1024>(sum, &all);
#pragma unroll
        for (uint32_t i = 0; i < 8; i++) {
            const uint32_t x = c0 + threadIdx.x * 8 + i;
            if (x < ntiles) row[x] = run;
            run += v[i];
        }
        carry += (uint32_t)all;
    }
    if (threadIdx.x == 0) tot[blockIdx.x] = carry;
}

template <uint32_t NT, uint32_t ITEMS, typename In>
__global__ __launch_bounds__(NT) void k_key_scatter(In in, uint64_t *out, int shift, int bits, uint32_t n,
                                                    uint32_t ntiles, const uint32_t *offs, const uint32_t *tot) {
    constexpr uint32_t NW = NT / 64, TILE = NT * ITEMS;
    static_assert(NT >= KS_BINS, "a thread per digit");
    __shared__ uint64_t s_k[TILE];
    __shared__ uint32_t s_wh[NW][KS_BINS];  // a wave's keys per digit, then its first place in the tile
    __shared__ uint32_t s_gb[KS_BINS];      // output place of the tile's place 0 as seen from a digit
    const uint32_t t = threadIdx.x, w = t >> 6, lane = lane_id(), mask = (1u << bits) - 1;
    const uint64_t base = (uint64_t)blockIdx.x * TILE;
    const uint32_t cnt = n - base < TILE ? (uint32_t)(n - base) : TILE;
    // the tile's first place per digit, loaded early
    uint32_t tg = 0, tt = 0;
    if (t <= mask) {
        tg = offs[(uint64_t)t * ntiles + blockIdx.x];
        tt = tot[t];
    }
    uint64_t k[ITEMS];
    uint32_t rk[ITEMS];
    const uint32_t wbase = w * 64 * ITEMS;
#pragma unroll
    for (uint32_t i = 0; i < ITEMS; i++) {
        const uint32_t q = wbase + i * 64 + lane;
        k[i] = in((uint32_t)(base + (q < cnt ? q : cnt - 1)));
    }
#pragma unroll
    for (uint32_t q = 0; q < KS_BINS / 64; q++) s_wh[w][q * 64 + lane] = 0;
    // ranks within the wave, in input order (round, lane); a wave's LDS
    // accesses run in program order, which the volatile pointer keeps
    volatile uint32_t *wh = s_wh[w];
#pragma unroll
    for (uint32_t i = 0; i < ITEMS; i++) {
        const bool valid = wbase + i * 64 + lane < cnt;
        const uint32_t d = (uint32_t)(k[i] >> shift) & mask;
        const uint64_t peers = digit_peers(d, bits, valid);
        const uint32_t before = rank_below(peers);
        const uint32_t old = wh[d];
        rk[i] = old + before;
        if (valid && before == 0) wh[d] = old + (uint32_t)__popcll(peers);
    }
    __syncthreads();
    {
        // digit t: its keys per wave -> places, its start in the tile and its
        // start in the output (two exclusive scans over the digits in one)
        uint32_t run = 0;
        if (t < KS_BINS)
#pragma unroll
            for (uint32_t q = 0; q < NW; q++) {
                const uint32_t c = s_wh[q][t];
                s_wh[q][t] = run;
                run += c;
            }
        uint64_t all;
        const uint64_t ex = block_exclusive_sum<NT>(((uint64_t)tt << 32) | run, &all);
        const uint32_t start = (uint32_t)ex;
        if (t < KS_BINS) {
            s_gb[t] = (uint32_t)(ex >> 32) + tg - start;
#pragma unroll
            for (uint32_t q = 0; q < NW; q++) s_wh[q][t] += start;
        }
    }
    __syncthreads();
#pragma unroll
    for (uint32_t i = 0; i < ITEMS; i++)
        if (wbase + i * 64 + lane < cnt) s_k[s_wh[w][(uint32_t)(k[i] >> shift) & mask] + rk[i]] = k[i];
    __syncthreads();
#pragma unroll
    for (uint32_t i = 0; i < ITEMS; i++) {
        const uint32_t p = i * NT + t;
        if (p < cnt) {
            const uint64_t key = s_k[p];
            const uint32_t at = s_gb[(uint32_t)(key >> shift) & mask] + p;
            if (at < n) out[at] = key;  // always, when the histogram matches
        }
    }
}

template <uint32_t NT, uint32_t ITEMS, typename In>
static void key_pass(gsi_ctx *c, In in, uint64_t *out, int shift, int bits, uint32_t n, uint32_t *hist, uint32_t *tot,
                     double in_bytes) {
    const uint32_t ntiles = (uint32_t)(((uint64_t)n + NT * ITEMS - 1) / (NT * ITEMS));
    launch(c, "k_radix_hist", in_bytes * n, k_key_hist<NT, ITEMS, In>, ntiles, NT, in, shift, bits, n, ntiles, hist);
    launch(c, "k_radix_offsets", 8.0 * ntiles * (1u << bits), k_key_offsets, 1u << bits, 1024, hist, ntiles, tot);
    launch(c, "k_radix_scatter", (in_bytes + 8.0) * n, k_key_scatter<NT, ITEMS, In>, ntiles, NT, in, out, shift, bits,
           n, ntiles, (const uint32_t *)hist, (const uint32_t *)tot);
}

// Keys from which a tile holds 8192 keys (runs of 32 keys a digit); fewer
// keys take tiles of 2048, four times the workgroups, so that a few million
// keys still fill the chip.
constexpr uint32_t KS_WIDE = 1u << 23;

static uint32_t key_tiles(uint32_t n) {
    const uint32_t tile = n >= KS_WIDE ? 8192u : 2048u;
    return (uint32_t)(((uint64_t)n + tile - 1) / tile);
}

template <typename In>
static void key_pass_any(gsi_ctx *c, In in, uint64_t *out, int shift, int bits, uint32_t n, uint32_t *hist,
                         uint32_t *tot, double in_bytes) {
    if (n >= KS_WIDE) key_pass<512, 16>(c, in, out, shift, bits, n, hist, tot, in_bytes);
    else key_pass<256, 8>(c, in, out, shift, bits, n, hist, tot, in_bytes);
}

// passes over bits [lo, hi), as even as possible
static std::vector<std::pair<int, int>> key_passes(int lo, int hi) {
    std::vector<std::pair<int, int>> p;
    int np = (hi - lo + 7) / 8;
    for (int at = lo; np > 0; np--) {
        const int b = (hi - at + np - 1) / np;
        p.push_back({at, b});
        at += b;
    }
    return p;
}

bool key_sort(gsi_ctx *c, uint32_t n, uint64_t *a, uint64_t *tmp, int lo, int hi, Scratch &s) {
    if (n <= 1 || hi <= lo) return false;
    uint32_t *hist = s.get<uint32_t>((uint64_t)KS_BINS * key_tiles(n), "radix histogram");
    uint32_t *tot = s.get<uint32_t>(KS_BINS, "radix digit totals");
    bool in_tmp = false;
    for (auto &p : key_passes(lo, hi)) {
        key_pass_any(c, KeyArray{in_tmp ? tmp : a}, in_tmp ? a : tmp, p.first, p.second, n, hist, tot, 8.0);
        in_tmp = !in_tmp;
    }
    s.drop(tot);
    s.drop(hist);
    return in_tmp;
}

bool edge_key_sort(gsi_ctx *c, uint32_t m, const uint32_t *src, const uint32_t *dst, const uint32_t *el, int vb,
                   uint64_t *a, uint64_t *tmp, Scratch &s) {
    const uint32_t n = 2 * m;
    uint32_t *hist = s.get<uint32_t>((uint64_t)KS_BINS * key_tiles(n), "radix histogram");
    uint32_t *tot = s.get<uint32_t>(KS_BINS, "radix digit totals");
    // the first pass packs the entries itself
    const auto passes = key_passes(0, 2 * vb);
    key_pass_any(c, EdgeKeys{src, dst, el, vb}, a, passes[0].first, passes[0].second, n, hist, tot, 6.0);
    bool in_tmp = false;
    for (size_t i = 1; i < passes.size(); i++) {
        key_pass_any(c, KeyArray{in_tmp ? tmp : a}, in_tmp ? a : tmp, passes[i].first, passes[i].second, n, hist, tot,
                     8.0);
        in_tmp = !in_tmp;
    }
    s.drop(tot);
    s.drop(hist);
    return in_tmp;
}

// ------------------------------------------------------------ radix sort
// Tiles of 4096 tuples (256 threads x 16 rounds).  Stability: within a tile
// tuple r*256 + t is handled in round r by thread t, so (round, wave, lane)
// is the input order; ranks are counted in that order.
constexpr int RS_THREADS = 256;
constexpr int RS_ROUNDS = 16;
constexpr int RS_TILE = RS_THREADS * RS_ROUNDS;

__global__ __launch_bounds__(RS_THREADS) void k_radix_hist(const uint32_t *key, int shift, uint32_t n,
                                                          uint32_t ntiles, uint32_t *hist) {
    __shared__ uint32_t h[256];
    h[threadIdx.x] = 0;
    __syncthreads();
    uint64_t base = (uint64_t)blockIdx.x * RS_TILE;
    for (int r = 0; r < RS_ROUNDS; r++) {
        uint64_t idx = base + (uint64_t)r * RS_THREADS + threadIdx.x;
        bool valid = idx < n;
        uint32_t d = valid ? (key[idx] >> shift) & 255u : 0u;
        uint64_t peers = digit_peers(d, 8, valid);
        if (valid && rank_below(peers) == 0) atomicAdd(&h[d], (uint32_t)__popcll(peers));
    }
    __syncthreads();
    hist[(uint64_t)threadIdx.x * ntiles + blockIdx.x] = h[threadIdx.x];
}

struct Arrays3 {
    uint32_t *p[3];
};

__global__ __launch_bounds__(RS_THREADS) void k_radix_scatter(Arrays3 src, Arrays3 dst, int key_arr, int shift,
                                                             uint32_t n, uint32_t ntiles, const uint64_t *offs) {
    __shared__ uint64_t s_goff[256];
    __shared__ uint32_t s_run[256];
    __shared__ uint32_t s_wc[RS_THREADS / 64][256];
    const uint32_t t = threadIdx.x, w = t >> 6;
    s_goff[t] = offs[(uint64_t)t * ntiles + blockIdx.x];
    s_run[t] = 0;
    const uint32_t *key = src.p[key_arr];
    uint64_t base = (uint64_t)blockIdx.x * RS_TILE;
    for (int r = 0; r < RS_ROUNDS; r++) {
#pragma unroll
        for (int q = 0; q < RS_THREADS / 64; q++) s_wc[q][t] = 0;
        __syncthreads();
        uint64_t idx = base + (uint64_t)r * RS_THREADS + t;
        bool valid = idx < n;
        uint32_t vals[3];
#pragma unroll
        for (int i = 0; i < 3; i++) vals[i] = valid ? src.p[i][idx] : 0u;
        uint32_t d = valid ? (key[idx] >> shift) & 255u : 0u;
        uint64_t peers = digit_peers(d, 8, valid);
        uint32_t rk = rank_below(peers);
        if (valid && rk == 0) s_wc[w][d] = (uint32_t)__popcll(peers);
        __syncthreads();
        {
            uint32_t run = s_run[t];
#pragma unroll
            for (int q = 0; q < RS_THREADS / 64; q++) {
                uint32_t cnt = s_wc[q][t];
                s_wc[q][t] = run;
                run += cnt;
            }
            s_run[t] = run;
        }
        __syncthreads();
        if (valid) {
            uint64_t pos = s_goff[d] + s_wc[w][d] + rk;
            if (pos >= n) pos = n - 1;  // unreachable when the histogram matches; never write out of bounds
#pragma unroll
            for (int i = 0; i < 3; i++) dst.p[i][pos] = vals[i];
        }
        __syncthreads();
    }
}

bool radix_sort(gsi_ctx *c, uint32_t n, uint32_t *const *a, uint32_t *const *tmp, const std::vector<SortPass> &passes,
                Scratch &s) {
    if (n <= 1 || passes.empty()) return false;
    uint32_t ntiles = (uint32_t)(((uint64_t)n + RS_TILE - 1) / RS_TILE);
    uint64_t nh = 256ull * ntiles;
    uint32_t *hist = s.get<uint32_t>(nh, "radix histogram");
    uint64_t *offs = s.get<uint64_t>(nh + 1, "radix offsets");
    Arrays3 A{}, B{};
    for (int i = 0; i < 3; i++) {
        A.p[i] = a[i];
        B.p[i] = tmp[i];
    }
    bool in_tmp = false;
    for (const SortPass &p : passes) {
        Arrays3 from = in_tmp ? B : A, to = in_tmp ? A : B;
        const uint32_t *key = from.p[p.key_arr];
        launch(c, "k_radix_hist", 4.0 * n, k_radix_hist, ntiles, RS_THREADS, key, p.shift, n, ntiles, hist);
        exclusive_scan(c, hist, nh, offs, s);
        launch(c, "k_radix_scatter", 24.0 * n, k_radix_scatter, ntiles, RS_THREADS, from, to, p.key_arr, p.shift, n,
               ntiles, (const uint64_t *)offs);
        in_tmp = !in_tmp;
    }
    s.drop(offs);
    s.drop(hist);
    return in_tmp;
}

}  // namespace gsi
