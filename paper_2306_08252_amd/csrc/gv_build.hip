// gv_build.hip -- bulk build (graph_init), canonical dump, adjacency read,
// structural audit.
//
// Bulk build (Sec. 4.3 initialisation and the "bulk" batch of Sec. 5.2): the
// COO list is sorted by (src, dst) with the radix sort, duplicates are
// dropped, each vertex's degree is read off the run boundaries, and one scan
// over the dictionary assigns every vertex a contiguous run of blocks and, if
// it needs two or more blocks, a power-of-two directory segment.  The pool is
// then exactly a CSR layout padded to whole blocks, written with coalesced
// stores.
#include <algorithm>
#include <chrono>
#include <cstddef>

#include "gv_graph.h"
#include "gv_prim.h"

namespace gv {

__device__ __forceinline__ uint64_t tidx() { return (uint64_t)blockIdx.x * kThreads + threadIdx.x; }
__device__ __forceinline__ uint32_t gwave() {
    return (uint32_t)(((uint64_t)blockIdx.x * kThreads + threadIdx.x) >> 6);
}

void read_counters(gv_graph* g) {
    static_assert(sizeof(DevCounters) % 16 == 0, "copied by the short way");
    hip_check(hipMemcpyAsync(g->hctr, g->v.ctr, sizeof(DevCounters), hipMemcpyDeviceToHost,
                             g->ctx.stream),
              "hipMemcpyAsync counters");
    hip_check(hipStreamSynchronize(g->ctx.stream), "hipStreamSynchronize");
    g->edge_bound_host = g->hctr->live_edges;
}

// Every counter but the stripes into pinned host memory, then the number of
// this read, which tells the host that they have arrived.
constexpr auto kStatSpin = std::chrono::milliseconds(1);
constexpr uint32_t kCtrHead = offsetof(DevCounters, stripe) / 4;
constexpr uint32_t kCtrTail = (offsetof(DevCounters, stripe) + sizeof(DevCounters::stripe)) / 4;
__global__ __launch_bounds__(kThreads) void k_export(const DevCounters* ctr, HostCounters* host,
                                                     unsigned long long number) {
    const uint32_t* from = (const uint32_t*)ctr;
    uint32_t* to = (uint32_t*)&host->c;
    for (uint32_t i = threadIdx.x; i < kCtrHead; i += kThreads) to[i] = from[i];
    for (uint32_t i = kCtrTail + threadIdx.x; i < sizeof(DevCounters) / 4; i += kThreads)
        to[i] = from[i];
    __threadfence_system();
    __syncthreads();
    if (threadIdx.x == 0)
        __hip_atomic_store(&host->number, number, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// For calls that wait for a batch's statistics and hand out nothing else: a
// copy and a stream synchronisation cost such a call 4 us more at 10^3 pairs and
// 17 at 10^5.  The wait gives up on a long queue (or one that failed) and
// synchronises.
void read_stats(gv_graph* g) {
    HostCounters* h = g->hmem;
    const unsigned long long number = ++g->stat_reads;
    hipLaunchKernelGGL(k_export, dim3(1), dim3(kThreads), 0, g->ctx.stream,
                       (const DevCounters*)g->v.ctr, h, number);
    hip_check(hipGetLastError(), "export counters");
    const auto start = std::chrono::steady_clock::now();
    for (uint32_t i = 1;; ++i) {
        if (__atomic_load_n(&h->number, __ATOMIC_ACQUIRE) == number) break;
        if (i % 64 == 0 && std::chrono::steady_clock::now() - start > kStatSpin) {
            hip_check(hipStreamSynchronize(g->ctx.stream), "hipStreamSynchronize");
            break;
        }
        __builtin_ia32_pause();
    }
    g->edge_bound_host = g->hctr->live_edges;
}

// Sort n keys of `bits` bits (n >= 2) with the one-sweep radix sort; `state`
// holds os_words(n, bits) words.  Synchronous: raises GV_EDEVICE if a
// look-back did not complete.  Returns true if the result is in k1.
static bool sort_keys(gv_graph* g, uint64_t* k0, uint64_t* k1, uint64_t n, int bits,
                      uint32_t* state) {
    Ctx& c = g->ctx;
    DevCounters* ctr = g->v.ctr;
    set_u32(g, &ctr->sort_n, (uint32_t)n);
    set_u32(g, &ctr->sort_err, 0);
    const bool flip = onesweep<uint64_t, false>(c, k0, k1, nullptr, nullptr, &ctr->sort_n, n,
                                                bits, state, &ctr->sort_err);
    read_counters(g);
    if (g->hctr->sort_err) fail(GV_EDEVICE, "sort look-back did not complete");
    return flip;
}

// ------------------------------------------------------------------ init
__global__ __launch_bounds__(kThreads) void k_init_active(GraphView g, uint64_t n_active) {
    const uint64_t v = tidx();
    const uint64_t words = (g.n_cap + 31) / 32;
    if (v < words) {
        const uint64_t lo = v * 32;
        uint32_t w = 0;
        if (n_active >= lo + 32) w = 0xffffffffu;
        else if (n_active > lo) w = (1u << (n_active - lo)) - 1u;
        g.active[v] = w;
    }
}

// keys of the initial edges with the sort's digit counts (per workgroup); an
// id out of range raises a flag (a plain store, taken only on error) that the
// host checks before any id is used as an index
__global__ __launch_bounds__(kOsThreads) void k_init_pack(GraphView g, const uint32_t* src,
                                                          const uint32_t* dst, uint64_t m,
                                                          uint64_t n, int passes, uint64_t* keys,
                                                          uint32_t* hpart) {
    __shared__ uint32_t h[kOsHistCopies][8][kRadix];
    const uint32_t t = threadIdx.x;
    for (int i = t; i < kOsHistCopies * 8 * kRadix; i += kOsThreads) (&h[0][0][0])[i] = 0;
    __syncthreads();
    const uint32_t copy = kOsHistCopies == 1 ? 0u : (t >> 6) & (kOsHistCopies - 1);
    bool bad = false;
    const uint64_t ntiles = (m + kHistTile - 1) / kHistTile;
    for (uint64_t tl = blockIdx.x; tl < ntiles; tl += gridDim.x) {
        const uint64_t i = tl * kHistTile + t;
        if (i >= m) continue;
        const uint32_t su = src[i], du = dst[i];
        bad |= ((uint64_t)su >= n) | ((uint64_t)du >= n);
        const uint64_t key = ((uint64_t)su << g.L) | du;
        keys[i] = key;
        for (int p = 0; p < passes; ++p)
            atomicAdd(&h[copy][p][(uint32_t)(key >> (p * kRadixBits)) & (kRadix - 1)], 1u);
    }
    if (bad) g.ctr->vany = 1;
    __syncthreads();
    uint32_t* out = hpart + (uint64_t)blockIdx.x * passes * kRadix;
    for (int i = t; i < passes * kRadix; i += kOsThreads) {
        uint32_t x = 0;
#pragma unroll
        for (int c = 0; c < kOsHistCopies; ++c) x += h[c][i / kRadix][i % kRadix];
        out[i] = x;
    }
}

// Scan over the sorted keys: first occurrences in the low half, first
// occurrences of a source in the high half.  The sink compacts the distinct
// keys and writes each source's run of them, [run[v].x, run[v].y): a source's
// first key ends the run before it.
struct FirstIn {
    const uint64_t* keys;
    uint32_t L;
    struct Rec {
        uint64_t k, p;
    };
    __device__ uint64_t limit(uint64_t m) const { return m; }
    __device__ Rec load(uint64_t i, bool) const { return Rec{keys[i], keys[i ? i - 1 : 0]}; }
    __device__ void deref(Rec&) const {}
    __device__ unsigned long long value(uint64_t i, const Rec& r) const {
        const unsigned long long first = i == 0 || r.k != r.p;
        const unsigned long long head = i == 0 || (r.k >> L) != (r.p >> L);
        return first | (head << 32);
    }
};

struct FirstOut {
    uint32_t L;
    uint64_t* ukeys;
    uint2* run;
    __device__ void operator()(uint64_t i, const FirstIn::Rec& r, uint64_t m,
                               unsigned long long pre) const {
        const uint32_t pos = (uint32_t)pre;
        const bool first = i == 0 || r.k != r.p;
        if (first) ukeys[pos] = r.k;
        if (i == 0 || (r.k >> L) != (r.p >> L)) {
            run[r.k >> L].x = pos;
            if (i) run[r.p >> L].y = pos;
        }
        if (i + 1 == m) run[r.k >> L].y = pos + (first ? 1u : 0u);
    }
};

// per vertex: blocks in the low half, directory entries in the high half
struct LayoutIn {
    GraphView g;
    const uint2* run;
    __device__ unsigned long long operator()(uint64_t v) const {
        if (v >= g.n_cap) return 0ull;
        const uint2 r = run[v];
        const uint32_t nb = nblocks(g, r.y - r.x);
        const unsigned long long de = nb >= 2 ? (1ull << ceil_log2(nb)) : 0ull;
        return (unsigned long long)nb | (de << 32);
    }
};

__global__ __launch_bounds__(kThreads) void k_init_layout(GraphView g, const uint2* run,
                                                          const unsigned long long* off) {
    const uint64_t v = tidx();
    if (v >= g.n_cap) return;
    const uint2 q = run[v];
    VRec r{q.y - q.x, 0u, kNoDir, 0u};
    const uint32_t nb = nblocks(g, r.deg);
    if (nb == 1) {
        r.dir = (uint32_t)off[v];
    } else if (nb) {
        r.dir = (uint32_t)(off[v] >> 32);
        r.dcls = ceil_log2(nb);
    }
    g.vt[v] = r;
}

// scatter: edge p of the sorted unique list goes to slot (p - run start) of
// its vertex's contiguous blocks; a block's first edge also writes the
// block's owner record and directory entry (a thread per vertex that wrote
// them took 200 us on R-MAT 2^20 / 2^24: the longest adjacency has 4096
// blocks)
__global__ __launch_bounds__(kThreads) void k_init_scatter(GraphView g, const uint64_t* ukeys,
                                                           const uint2* run,
                                                           const unsigned long long* off,
                                                           uint64_t mu) {
    const uint64_t p = tidx();
    if (p >= mu) return;
    const uint64_t k = ukeys[p];
    const uint32_t v = (uint32_t)(k >> g.L);
    const uint2 q = run[v];
    const unsigned long long o = off[v];
    const uint32_t s = (uint32_t)p - q.x;
    const uint32_t j = s >> g.log2B, blk = (uint32_t)o + j;
    const uint64_t a = ((uint64_t)blk << g.log2B) + (s & (g.B - 1));
    g.pool[a] = (uint32_t)(k & ((1ull << g.L) - 1));
    attr_zero(g, a);
    if ((s & (g.B - 1)) == 0) {
        g.bown[blk] = make_uint2(v, j);
        if (q.y - q.x > g.B) g.dir[(o >> 32) + j] = blk;
    }
}

__global__ void k_init_counters(GraphView g, unsigned long long blocks, unsigned long long dents,
                                unsigned long long edges) {
    DevCounters* c = g.ctr;
    c->live_edges = edges;
    c->free_cnt = 0;
    c->bump = blocks;
    c->dir_bump = dents;
    c->dir_live = dents;
    for (int k = 0; k < kMaxClass; ++k) {
        c->dfree_cnt[k] = 0;
        c->dreq[k] = 0;
    }
    c->err_batch = c->err_sticky = 0;
}

static uint32_t paper_block_rule(uint64_t edges, uint64_t nonzero) {
    // Sec. 4.3: average degree of the non-zero-degree vertices of the first
    // batch, rounded up to a power of two and kept within [8, 64].
    if (edges == 0 || nonzero == 0) return 8;
    uint64_t avg = (edges + nonzero - 1) / nonzero;
    uint64_t b = 1;
    while (b < avg) b <<= 1;
    return (uint32_t)std::min<uint64_t>(64, std::max<uint64_t>(8, b));
}

void bulk_build(gv_graph* g, uint64_t n, const uint32_t* src, const uint32_t* dst, uint64_t m,
                const gv_config& cfg) {
    Ctx& c = g->ctx;
    GraphView& v = g->v;
    c.launch("init_active", k_init_active, div_up((v.n_cap + 31) / 32, kThreads), kThreads, v, n);
    set_u32(g, &v.ctr->vany, 0);

    const int bits = 2 * (int)v.L;
    uint64_t mu = 0, nonzero = 0;
    struct Arr {
        uint64_t* k0;
        uint64_t* k1;
        unsigned long long* part;
        uint32_t* state;
        unsigned long long* off;
        unsigned long long* part64;
        uint2* run;
    } A{};
    const bool sorts = m > 1 && bits > 0;
    const uint64_t state_words = sorts ? os_words(m, bits) : 0;
    auto carve = [&](Carver& cv) {
        A.k0 = cv.take<uint64_t>(std::max<uint64_t>(m, 1));
        A.k1 = cv.take<uint64_t>(std::max<uint64_t>(m, 1));
        A.part = cv.take<unsigned long long>(scan2_parts(m));
        // (a single key's digits are counted too, for no pass)
        A.state = cv.take<uint32_t>(std::max<uint64_t>(state_words, 8 * kRadix));
        A.off = cv.take<unsigned long long>(v.n_cap + 1);
        A.part64 = cv.take<unsigned long long>(scan_partials_needed(v.n_cap + 1));
        A.run = cv.take<uint2>(v.n_cap);
    };
    {
        Carver mz(nullptr);
        carve(mz);
        g->scratch.ensure(mz.used, c.stream);
        Carver cv(g->scratch.ptr);
        carve(cv);
    }
    uint64_t* ukeys = nullptr;
    zero_words(c, (uint32_t*)A.run, 2 * v.n_cap);
    if (m > 0) {
        if (m >= kOsMaxKeys) fail(GV_EINVAL, "2^30 or more edges");
        const int passes = sorts ? os_passes(bits) : 0;
        if (sorts) zero_words(c, A.state, os_zero_words(m, bits));
        c.launch("init_pack", k_init_pack, os_hist_groups(m), kOsThreads, v, src, dst, m, n,
                 passes, A.k0, sorts ? os_hpart(A.state, m, bits) : A.state);
        bool flip = false;
        if (sorts) {
            set_u32(g, &v.ctr->sort_err, 0);
            os_hist_sum(c, A.state, m, bits, nullptr, nullptr, nullptr, nullptr);
            flip = onesweep_passes<uint64_t, false>(c, A.k0, A.k1, nullptr, nullptr, nullptr, m,
                                                    bits, A.state, &v.ctr->sort_err);
        }
        read_counters(g);
        if (g->hctr->vany) fail(GV_ERANGE, "edge id >= num_vertices");
        if (sorts && g->hctr->sort_err) fail(GV_EDEVICE, "sort look-back did not complete");
        uint64_t* keys = flip ? A.k1 : A.k0;
        ukeys = flip ? A.k0 : A.k1;
        scan2(c, "init_unique", FirstIn{keys, v.L}, FirstOut{v.L, ukeys, A.run}, m, A.part,
              &v.ctr->edges);
        read_counters(g);
        if (g->hctr->err_wait) fail(GV_EDEVICE, "a scan's wait ran out");
        mu = g->hctr->edges & 0xffffffffull;
        nonzero = g->hctr->edges >> 32;
    }
    uint32_t B = cfg.block_slots ? cfg.block_slots : paper_block_rule(mu, nonzero);
    v.B = B;
    v.log2B = log2_exact(B);

    scan_excl<unsigned long long>(c, LayoutIn{v, A.run}, ArrOut<unsigned long long>{A.off},
                                  v.n_cap + 1, A.part64, &v.ctr->edges);
    read_counters(g);
    const uint64_t blocks = g->hctr->edges & 0xffffffffull;
    const uint64_t dents = g->hctr->edges >> 32;

    // pool and directory sizing
    uint64_t cap_blocks = cfg.pool_bytes ? cfg.pool_bytes / (4ull * B) : 2 * blocks + (1ull << 20);
    cap_blocks = std::min<uint64_t>(cap_blocks, 0xfffffff0ull);
    if (blocks > cap_blocks) fail(GV_ENOMEM, "pool too small for the initial graph");
    uint64_t dir_cap = cfg.directory_entries ? cfg.directory_entries
                                             : 4 * cap_blocks + (1ull << 20);
    dir_cap = std::min<uint64_t>(dir_cap, 0xfffffff0ull);
    if (dents > dir_cap) fail(GV_ENOMEM, "directory too small for the initial graph");
    uint64_t dfree_total = 0;
    for (int k = 0; k < kMaxClass; ++k) {
        v.dfree_base[k] = dfree_total;
        dfree_total += (k == 0) ? 0 : (dir_cap >> k);
    }
    // one allocation: pool, free list, block owners, directory, its free
    // lists, attributes
    auto carve_pool = [&](Carver& cv) {
        v.pool = cv.take<uint32_t>(std::max<uint64_t>(cap_blocks * B, 1));
        v.free_stack = cv.take<uint32_t>(std::max<uint64_t>(cap_blocks, 1));
        v.bown = cv.take<uint2>(std::max<uint64_t>(cap_blocks, 1));
        v.dir = cv.take<uint32_t>(std::max<uint64_t>(dir_cap, 1));
        v.dfree = cv.take<uint32_t>(std::max<uint64_t>(dfree_total, 1));
        v.apool = v.A ? cv.take<uint32_t>(cap_blocks * B * v.A) : nullptr;
    };
    Carver mp(nullptr);
    carve_pool(mp);
    dev_malloc(&g->mem_pool, mp.used, "hipMalloc pool");
    Carver cp(g->mem_pool);
    carve_pool(cp);
    v.cap_blocks = cap_blocks;
    v.dir_cap = dir_cap;
    g->item_slots = cap_blocks * B;

    c.launch("init_layout", k_init_layout, div_up(v.n_cap, kThreads), kThreads, v,
             (const uint2*)A.run, (const unsigned long long*)A.off);
    if (mu > 0)
        c.launch("init_scatter", k_init_scatter, div_up(mu, kThreads), kThreads, v,
                 (const uint64_t*)ukeys, (const uint2*)A.run,
                 (const unsigned long long*)A.off, mu);
    c.launch("init_counters", k_init_counters, 1, 1, v, (unsigned long long)blocks,
             (unsigned long long)dents, (unsigned long long)mu);
    hip_check(hipStreamSynchronize(c.stream), "hipStreamSynchronize");
    g->edge_bound_host = mu;
}

// ------------------------------------------------------------------ dump
struct DegIn {
    GraphView g;
    __device__ unsigned long long operator()(uint64_t v) const {
        return v < g.n_cap ? g.vt[v].deg : 0ull;
    }
};

// Sums of a dump, striped over 64 lines (the host adds them up).
constexpr int kStripeSum = 2, kStripeEdges = 3;

// Classes of rows by degree: a dump orders rows of up to kRowLane entries by
// 16 lanes each, and up to kRowMid by a wave in registers.  Longer rows are
// listed and ordered by workgroups, as bitmaps of the destinations where the
// table is small enough, else up to kRowBig entries in LDS and longer ones by
// the one-sweep sort as (row, destination) keys.
constexpr uint32_t kRowLane = 16, kRowMid = 1024, kRowBig = 16384;
enum { kRowsBig = 0, kRowsHuge = 1, kHugeEdges = 2 };

// Clears the sums and counts the rows past kRowMid by class (and the entries
// of the longest), for the host to size their lists.
__global__ __launch_bounds__(kThreads) void k_dump_begin(GraphView g) {
    DevCounters* c = g.ctr;
    const uint32_t t = threadIdx.x;
    if (t < 64) c->stripe[t][kStripeSum] = c->stripe[t][kStripeEdges] = 0ull;
    if (t < 4) {
        c->rows[t] = 0ull;
        c->row_at[t] = 0u;
    }
}

__global__ __launch_bounds__(kThreads) void k_dump_classes(GraphView g, uint32_t rowbig) {
    __shared__ unsigned long long lds[kWaves];
    unsigned long long big = 0, huge = 0, edges = 0;
    const uint64_t stride = (uint64_t)gridDim.x * kThreads;
    for (uint64_t v = tidx(); v < g.n_cap; v += stride) {
        const uint32_t d = g.vt[v].deg;
        big += d > kRowMid && d <= rowbig;
        huge += d > rowbig;
        edges += d > rowbig ? d : 0u;
    }
    big = block_sum(big, lds);
    huge = block_sum(huge, lds);
    edges = block_sum(edges, lds);
    if (threadIdx.x == 0) {
        if (big) atomicAdd(&g.ctr->rows[kRowsBig], big);
        if (huge) atomicAdd(&g.ctr->rows[kRowsHuge], huge);
        if (edges) atomicAdd(&g.ctr->rows[kHugeEdges], edges);
    }
}

// Count and checksum of the stored edges by a pass over the pool's handed-out
// blocks, a thread per slot of a block: the block's owner record names the
// vertex and index it was last given to, and it holds edges when that vertex
// still holds the block there.  Bound: HBM (4 B per slot, 8 B per block); the
// vertex records and directory entries of neighbouring blocks are neighbours
// after a bulk build.  A wave per vertex took 2320 us on R-MAT 2^20 / 2^24
// (the longest row, 65 thousand entries, was one wave's chain of loads); this
// pass takes 68.
__global__ __launch_bounds__(kThreads) void k_dump_checksum(GraphView g) {
    __shared__ unsigned long long lds[kWaves];
    unsigned long long h = 0, e = 0;
    const uint64_t n = (uint64_t)g.ctr->bump << g.log2B;
    const uint64_t stride = (uint64_t)gridDim.x * kThreads;
    for (uint64_t a = tidx(); a < n; a += stride) {
        const uint32_t b = (uint32_t)(a >> g.log2B);
        const uint2 ow = g.bown[b];
        const uint32_t x = g.pool[a];
        if (ow.x >= g.n_cap) continue;  // (never for a block handed out)
        const VRec r = g.vt[ow.x];
        if (ow.y >= nblocks(g, r.deg)) continue;
        const uint64_t s = ((uint64_t)ow.y << g.log2B) + (a & (g.B - 1));
        if (s >= r.deg || block_of(g, r, ow.y) != b) continue;
        h += mix64(((uint64_t)ow.x << 32) | x);
        ++e;
    }
    h = block_sum(h, lds);
    e = block_sum(e, lds);
    if (threadIdx.x == 0) {
        atomicAdd(&g.ctr->stripe[blockIdx.x & 63][kStripeSum], h);
        atomicAdd(&g.ctr->stripe[blockIdx.x & 63][kStripeEdges], e);
    }
}

// Bitonic networks in a wave's registers: element i = j * 64 + lane in x[j].
// A step of distance h < 64 exchanges lanes (data-parallel moves within 16
// lanes, row swaps for 16 and 32), one of h >= 64 exchanges registers; both
// are compile-time, so a step is three or four vector instructions per
// register.  (The same networks on LDS words took 17 instructions per
// compare-exchange in address arithmetic: 280 us for the rows of 65 to 1024
// entries of R-MAT 2^20 / 2^24.)
template <uint32_t H>
__device__ __forceinline__ void lane_minmax(uint32_t x, uint32_t& mn, uint32_t& mx) {
    if constexpr (H >= 16) {
        // both results hold the lower and the upper rows' values
        const auto r = H == 16 ? __builtin_amdgcn_permlane16_swap(x, x, false, false)
                               : __builtin_amdgcn_permlane32_swap(x, x, false, false);
        mn = min((uint32_t)r[0], (uint32_t)r[1]);
        mx = max((uint32_t)r[0], (uint32_t)r[1]);
    } else {
        uint32_t y;
        if constexpr (H == 1) y = __builtin_amdgcn_update_dpp(0u, x, 0xB1, 0xf, 0xf, true);
        else if constexpr (H == 2) y = __builtin_amdgcn_update_dpp(0u, x, 0x4E, 0xf, 0xf, true);
        else if constexpr (H == 4) y = __builtin_amdgcn_ds_swizzle(x, (4 << 10) | 0x1f);
        else y = __builtin_amdgcn_update_dpp(0u, x, 0x128, 0xf, 0xf, true);
        mn = min(x, y);
        mx = max(x, y);
    }
}

// the steps of distance H, H / 2, ... 1 of the merge of runs of K elements
template <uint32_t E, uint32_t K, uint32_t H>
__device__ __forceinline__ void wave_merge(uint32_t (&x)[E], uint32_t lane) {
    if constexpr (H >= 64) {
        constexpr uint32_t hj = H / 64;
#pragma unroll
        for (uint32_t j = 0; j < E; ++j) {
            if (j & hj) continue;
            const uint32_t a = min(x[j], x[j + hj]), b = max(x[j], x[j + hj]);
            const bool up = ((j * 64) & K) == 0;
            x[j] = up ? a : b;
            x[j + hj] = up ? b : a;
        }
    } else {
#pragma unroll
        for (uint32_t j = 0; j < E; ++j) {
            uint32_t mn, mx;
            lane_minmax<H>(x[j], mn, mx);
            const bool up = K < 64 ? (lane & K) == 0 : ((j * 64) & K) == 0;
            x[j] = ((lane & H) == 0) == up ? mn : mx;
        }
    }
    if constexpr (H > 1) wave_merge<E, K, H / 2>(x, lane);
}

template <uint32_t E, uint32_t N, uint32_t K = 2>
__device__ __forceinline__ void wave_sort(uint32_t (&x)[E], uint32_t lane) {
    wave_merge<E, K, K / 2>(x, lane);
    if constexpr (K < N) wave_sort<E, N, K * 2>(x, lane);
}

// Bitonic sort of the m (a power of two) words at s by the nt threads of a
// workgroup.
__device__ __forceinline__ void lds_bitonic(uint32_t* s, uint32_t m, uint32_t t, uint32_t nt) {
    for (uint32_t k = 2; k <= m; k <<= 1) {
        for (uint32_t h = k >> 1; h > 0; h >>= 1) {
            __syncthreads();
            for (uint32_t c = t; c < m / 2; c += nt) {
                const uint32_t i = ((c & ~(h - 1)) << 1) | (c & (h - 1));
                const uint32_t a = s[i], b = s[i + h];
                if ((a > b) == ((i & k) == 0)) {
                    s[i] = b;
                    s[i + h] = a;
                }
            }
        }
    }
    __syncthreads();
}

// A row of up to E * 64 entries, in a wave's registers; returns the lane's
// share of the row's checksum.
template <uint32_t E>
__device__ __forceinline__ unsigned long long dump_row(const GraphView& g, uint64_t u,
                                                       const VRec& r, uint32_t lane,
                                                       uint32_t* out) {
    uint32_t x[E];
    unsigned long long h = 0;
#pragma unroll
    for (uint32_t j = 0; j < E; ++j)
        x[j] = g.pool[slot_addr(g, r, min(j * 64 + lane, r.deg - 1))];
#pragma unroll
    for (uint32_t j = 0; j < E; ++j) {
        const bool in = j * 64 + lane < r.deg;
        h += in ? mix64((u << 32) | x[j]) : 0ull;
        x[j] = in ? x[j] : kTomb;
    }
    wave_sort<E, E * 64>(x, lane);
#pragma unroll
    for (uint32_t j = 0; j < E; ++j)
        if (j * 64 + lane < r.deg) out[j * 64 + lane] = x[j];
    return h;
}

// Rows of up to kRowMid entries, ordered in registers and written at their CSR
// offsets: four vertices per wave per round, 16 lanes each; a row past
// kRowLane entries is taken by the whole wave.  Longer rows are listed by
// class (a few per thousand: listing the rows of 65 to 1024 entries as well,
// 50 thousand appends to one counter, took 300 us).  Adds up the checksum of
// the rows it writes.
__global__ __launch_bounds__(kThreads) void k_dump_rows(GraphView g,
                                                        const unsigned long long* offs,
                                                        uint32_t* out, uint32_t* big,
                                                        uint32_t* huge, uint32_t rowbig) {
    __shared__ unsigned long long lds[kWaves];
    const uint32_t lane = lane_id(), sub = lane & 15;
    unsigned long long h = 0;
    // A wave's place in a round turns by a large odd step from round to round:
    // with a plain stride (a power of two) one wave takes the vertices that
    // share their low bits, and on R-MAT tables the longest rows are those of
    // few set bits (1500 us instead of 255).
    const uint32_t nw = gridDim.x * kWaves, turn = (uint32_t)(nw * 0.618) | 1u;
    uint32_t at = gwave();
    for (uint64_t q0 = 0; q0 * 4 < g.n_cap; q0 += nw, at = (at + turn) % nw) {
        const uint64_t q = q0 + at;
        const uint64_t u = q * 4 + (lane >> 4);
        const bool live = u < g.n_cap;
        const VRec r = live ? g.vt[u] : VRec{0u, 0u, kNoDir, 0u};
        const uint32_t d = r.deg;
        const uint64_t off = live ? offs[u] : 0ull;
        uint32_t x[1] = {kTomb};
        if (d <= kRowLane && sub < d) {
            x[0] = g.pool[slot_addr(g, r, sub)];
            h += mix64((u << 32) | x[0]);
        }
        // (the last merge ascends in every group of 16)
        wave_sort<1, kRowLane / 2>(x, sub);
        wave_merge<1, 64, kRowLane / 2>(x, sub);
        if (d <= kRowLane && sub < d) out[off + sub] = x[0];
        const bool head = sub == 0;
        uint64_t m = ballot(head && d > kRowLane && d <= kRowMid);
        while (m) {
            const int l = __ffsll((unsigned long long)m) - 1;
            m &= m - 1;
            VRec w;
            w.deg = __builtin_amdgcn_readlane(r.deg, l);
            w.dir = __builtin_amdgcn_readlane(r.dir, l);
            w.dcls = __builtin_amdgcn_readlane(r.dcls, l);
            const uint64_t wu = q * 4 + ((uint32_t)l >> 4);
            uint32_t* wo = out + wave_read((unsigned long long)off, l);
            if (w.deg <= 64) h += dump_row<1>(g, wu, w, lane, wo);
            else if (w.deg <= 128) h += dump_row<2>(g, wu, w, lane, wo);
            else if (w.deg <= 256) h += dump_row<4>(g, wu, w, lane, wo);
            else if (w.deg <= 512) h += dump_row<8>(g, wu, w, lane, wo);
            else h += dump_row<16>(g, wu, w, lane, wo);
        }
        if (ballot(head && d > kRowMid)) {
            DevCounters* c = g.ctr;
            wave_append(head && d > kRowMid && d <= rowbig, (uint32_t)u, &c->row_at[kRowsBig],
                        big);
            wave_append(head && d > rowbig, (uint32_t)u, &c->row_at[kRowsHuge], huge);
        }
    }
    h = block_sum(h, lds);
    if (threadIdx.x == 0 && h) atomicAdd(&g.ctr->stripe[blockIdx.x & 63][kStripeSum], h);
}

// Rows past kRowMid entries on tables of up to 2^kWinMaxLog vertices: a
// workgroup per (row, window of 2^kWinLogBits destinations) marks the row's
// destinations of its window in an LDS bitmap and writes the set bits in
// order, after the row's destinations below the window (counted on the way).
// Bound: a sweep of the 128 KB bitmap and a pass over the row, whatever the
// row's length: 132 us for the 1350 rows of 1025 to 66 thousand entries of
// R-MAT 2^20 / 2^24, where an LDS bitonic network (225 us) and the one-sweep
// sort for rows past 16384 (100 us) took longer.  From 2^23 vertices on, with
// eight windows or more per row, the network is the shorter one.  Word w sits at w + w / 32,
// so that the 32 words of each thread start in different banks.
constexpr uint32_t kWinLogBits = 20, kWinMaxLog = 22;
constexpr uint32_t kWinWords = 1u << (kWinLogBits - 5);
constexpr uint32_t kWinThreads = 1024, kWinPer = kWinWords / kWinThreads;
static_assert(kWinPer == 32, "a padding word per thread");
__global__ __launch_bounds__(kWinThreads) void k_dump_rows_win(GraphView g,
                                                               const unsigned long long* offs,
                                                               uint32_t* out,
                                                               const uint32_t* list,
                                                               uint32_t rows, uint32_t nwin) {
    __shared__ uint32_t bm[kWinWords + kWinThreads];
    __shared__ uint32_t s_w[kWinThreads / 64], s_low;
    const uint32_t t = threadIdx.x, w = t >> 6;
    unsigned long long h = 0;
    for (uint64_t it = blockIdx.x; it < (uint64_t)rows * nwin; it += gridDim.x) {
        const uint32_t u = list[it / nwin], win = (uint32_t)(it % nwin);
        const VRec r = g.vt[u];
        uint32_t* o = out + offs[u];
        for (uint32_t i = t; i < kWinWords + kWinThreads; i += kWinThreads) bm[i] = 0u;
        if (t == 0) s_low = 0u;
        __syncthreads();
        uint32_t low = 0;
        constexpr uint32_t kU = 8;
        for (uint32_t s0 = t; s0 < r.deg; s0 += kU * kWinThreads) {
            uint32_t x[kU];
#pragma unroll
            for (uint32_t j = 0; j < kU; ++j)
                x[j] = g.pool[slot_addr(g, r, min(s0 + j * kWinThreads, r.deg - 1))];
#pragma unroll
            for (uint32_t j = 0; j < kU; ++j) {
                if (s0 + j * kWinThreads >= r.deg) continue;
                const uint32_t q = x[j] >> kWinLogBits;
                if (win == 0) h += mix64(((uint64_t)u << 32) | x[j]);
                low += q < win;
                if (q == win) {
                    const uint32_t b = x[j] & ((1u << kWinLogBits) - 1), wd = b >> 5;
                    atomicOr(&bm[wd + (wd >> 5)], 1u << (b & 31));
                }
            }
        }
        low = wave_sum(low);
        if (lane_id() == 0 && low) atomicAdd(&s_low, low);
        __syncthreads();
        uint32_t word[kWinPer], cnt = 0;
#pragma unroll
        for (uint32_t i = 0; i < kWinPer; ++i) {
            word[i] = bm[t * (kWinPer + 1) + i];
            cnt += __popc(word[i]);
        }
        const uint32_t inc = wave_incl_scan(cnt);
        if (lane_id() == 63) s_w[w] = inc;
        __syncthreads();
        uint32_t pos = s_low + inc - cnt;
        for (uint32_t i = 0; i < kWinThreads / 64; ++i) pos += i < w ? s_w[i] : 0u;
        const uint32_t v0 = (win << kWinLogBits) + t * kWinPer * 32;
#pragma unroll
        for (uint32_t i = 0; i < kWinPer; ++i) {
            uint32_t m = word[i];
            while (m) {
                const uint32_t b = __builtin_ctz(m);
                m &= m - 1;
                if (pos < r.deg) o[pos] = v0 + i * 32 + b;
                ++pos;
            }
        }
        __syncthreads();  // the words and sums are used again
    }
    h = wave_sum(h);
    if (lane_id() == 0 && h) atomicAdd(&g.ctr->stripe[(blockIdx.x + w) & 63][kStripeSum], h);
}

// Rows of kRowMid + 1 to kRowBig entries on larger tables: a workgroup each,
// a bitonic network on LDS words.
__global__ __launch_bounds__(kOsThreads) void k_dump_rows_big(GraphView g,
                                                              const unsigned long long* offs,
                                                              uint32_t* out, const uint32_t* list,
                                                              uint32_t rows) {
    __shared__ uint32_t s[kRowBig];
    const uint32_t t = threadIdx.x;
    unsigned long long h = 0;
    for (uint32_t k = blockIdx.x; k < rows; k += gridDim.x) {
        const uint64_t u = list[k];
        const VRec r = g.vt[u];
        const uint32_t d = min(r.deg, kRowBig);
        const uint64_t off = offs[u];
        uint32_t m = 2;
        while (m < d) m <<= 1;
        for (uint32_t i = t; i < m; i += kOsThreads) {
            uint32_t x = kTomb;
            if (i < d) {
                x = g.pool[slot_addr(g, r, i)];
                h += mix64((u << 32) | x);
            }
            s[i] = x;
        }
        lds_bitonic(s, m, t, kOsThreads);
        for (uint32_t i = t; i < d; i += kOsThreads) out[off + i] = s[i];
        __syncthreads();  // the next row reuses the words
    }
    h = wave_sum(h);
    if (lane_id() == 0 && h)
        atomicAdd(&g.ctr->stripe[(blockIdx.x + (t >> 6)) & 63][kStripeSum], h);
}

// Rows past kRowBig entries: their (row, destination) keys, kHugeParts
// workgroups per vertex; hoff[k] = entries of the rows before row k.
constexpr uint32_t kHugeParts = 64;
__global__ __launch_bounds__(kThreads) void k_dump_huge_offs(GraphView g, const uint32_t* huge,
                                                             uint32_t rows,
                                                             unsigned long long* hoff) {
    __shared__ unsigned long long lds[kWaves];
    unsigned long long carry = 0;
    for (uint32_t b = 0; b < rows; b += kThreads) {
        const uint32_t k = b + threadIdx.x;
        const unsigned long long d = k < rows ? g.vt[huge[k]].deg : 0u;
        unsigned long long tot;
        const unsigned long long ex = block_excl_scan(d, lds, tot);
        if (k < rows) hoff[k] = carry + ex;
        carry += tot;
    }
}

__global__ __launch_bounds__(kThreads) void k_dump_huge_gather(GraphView g, const uint32_t* huge,
                                                               uint32_t rows,
                                                               const unsigned long long* hoff,
                                                               uint64_t* keys) {
    unsigned long long h = 0;
    const uint32_t part = blockIdx.x % kHugeParts, rowg = gridDim.x / kHugeParts;
    for (uint32_t k = blockIdx.x / kHugeParts; k < rows; k += rowg) {
        const uint64_t u = huge[k];
        const VRec r = g.vt[u];
        for (uint64_t s = (uint64_t)part * kThreads + threadIdx.x; s < r.deg;
             s += (uint64_t)kHugeParts * kThreads) {
            const uint32_t x = g.pool[slot_addr(g, r, (uint32_t)s)];
            h += mix64((u << 32) | x);
            keys[hoff[k] + s] = ((uint64_t)k << g.L) | x;
        }
    }
    h = wave_sum(h);
    if (lane_id() == 0 && h) atomicAdd(&g.ctr->stripe[gwave() & 63][kStripeSum], h);
}

__global__ __launch_bounds__(kThreads) void k_dump_huge_out(GraphView g, const uint32_t* huge,
                                                            const unsigned long long* hoff,
                                                            const unsigned long long* offs,
                                                            const uint64_t* keys, uint64_t n,
                                                            uint32_t* out) {
    const uint64_t i = tidx();
    if (i >= n) return;
    const uint64_t key = keys[i];
    const uint32_t k = (uint32_t)(key >> g.L);
    out[offs[huge[k]] + (i - hoff[k])] = (uint32_t)(key & ((1ull << g.L) - 1));
}

// checksum and edge count added up over the stripes of the last counter read
static uint64_t stripe_sum(const gv_graph* g, int k) {
    uint64_t s = 0;
    for (int i = 0; i < 64; ++i) s += g->hctr->stripe[i][k];
    return s;
}

void dump(gv_graph* g, uint64_t* offsets, uint32_t* dst, uint64_t cap, uint64_t* checksum,
          uint64_t* edges) {
    Ctx& c = g->ctx;
    const GraphView& v = g->v;
    auto count_only = [&] {
        c.launch("dump_checksum", k_dump_checksum, resident_grid(k_dump_checksum, kThreads),
                 kThreads, v);
        read_counters(g);
        *checksum = stripe_sum(g, kStripeSum);
        *edges = stripe_sum(g, kStripeEdges);
    };
    c.launch("dump_begin", k_dump_begin, 1, kThreads, v);
    if (!dst || !offsets) return count_only();
    const bool win = v.L <= kWinMaxLog;  // no row is huge then
    const uint32_t rowbig = win ? 0xFFFFFFFFu : kRowBig;
    unsigned long long* offs = (unsigned long long*)offsets;
    unsigned long long* part = nullptr;
    {
        auto carve = [&](Carver& cv) {
            part = cv.take<unsigned long long>(scan_partials_needed(v.n_cap + 1));
        };
        Carver mz(nullptr);
        carve(mz);
        g->scratch.ensure(mz.used, c.stream);
        Carver cv(g->scratch.ptr);
        carve(cv);
    }
    scan_excl<unsigned long long>(c, DegIn{v}, ArrOut<unsigned long long>{offs}, v.n_cap + 1, part,
                                  &v.ctr->edges);
    c.launch("dump_classes", k_dump_classes,
             std::min<uint64_t>(div_up(v.n_cap, (uint64_t)kThreads * 4), 1024), kThreads, v,
             rowbig);
    read_counters(g);
    const uint64_t e = g->hctr->edges;
    *edges = e;
    if (cap < e) {
        count_only();
        fail(GV_ERANGE, "dump buffer too small");
    }
    if (e >= kOsMaxKeys) fail(GV_EINVAL, "2^30 or more edges");
    const uint64_t nbig = g->hctr->rows[kRowsBig];
    const uint64_t nhuge = g->hctr->rows[kRowsHuge], ehuge = g->hctr->rows[kHugeEdges];
    uint32_t *big = nullptr, *huge = nullptr, *state = nullptr;
    unsigned long long* hoff = nullptr;
    uint64_t *k0 = nullptr, *k1 = nullptr;
    const int bits = (int)v.L + (int)ceil_log2(std::max<uint64_t>(nhuge, 1));
    auto carve2 = [&](Carver& cv) {
        big = cv.take<uint32_t>(std::max<uint64_t>(nbig, 1));
        huge = cv.take<uint32_t>(std::max<uint64_t>(nhuge, 1));
        if (!nhuge) return;
        hoff = cv.take<unsigned long long>(nhuge);
        k0 = cv.take<uint64_t>(ehuge);
        k1 = cv.take<uint64_t>(ehuge);
        state = cv.take<uint32_t>(os_words(ehuge, bits));
    };
    {
        Carver mz(nullptr);
        carve2(mz);
        g->scratch.ensure(mz.used, c.stream);
        Carver cv(g->scratch.ptr);
        carve2(cv);
    }
    const unsigned long long* co = offs;
    c.launch("dump_rows", k_dump_rows,
             std::min<uint64_t>(div_up(v.n_cap, (uint64_t)kThreads / 16),
                                resident_grid(k_dump_rows, kThreads)),
             kThreads, v, co, dst, big, huge, rowbig);
    if (nbig && win) {
        const uint32_t nwin = v.L > kWinLogBits ? 1u << (v.L - kWinLogBits) : 1u;
        c.launch("dump_rows", k_dump_rows_win,
                 std::min<uint64_t>(nbig * nwin, resident_grid(k_dump_rows_win, kWinThreads)),
                 kWinThreads, v, co, dst, (const uint32_t*)big, (uint32_t)nbig, nwin);
    } else if (nbig) {
        c.launch("dump_rows", k_dump_rows_big,
                 std::min<uint64_t>(nbig, resident_grid(k_dump_rows_big, kOsThreads)), kOsThreads,
                 v, co, dst, (const uint32_t*)big, (uint32_t)nbig);
    }
    if (nhuge) {
        const uint32_t gy = (uint32_t)std::min<uint64_t>(nhuge, 1024);
        c.launch("dump_huge", k_dump_huge_offs, 1, kThreads, v, (const uint32_t*)huge,
                 (uint32_t)nhuge, hoff);
        c.launch("dump_huge", k_dump_huge_gather, (uint64_t)gy * kHugeParts, kThreads, v,
                 (const uint32_t*)huge, (uint32_t)nhuge, (const unsigned long long*)hoff, k0);
        const bool flip = sort_keys(g, k0, k1, ehuge, bits, state);
        c.launch("dump_huge", k_dump_huge_out, div_up(ehuge, kThreads), kThreads, v,
                 (const uint32_t*)huge, (const unsigned long long*)hoff, co,
                 (const uint64_t*)(flip ? k1 : k0), ehuge, dst);
    }
    read_counters(g);
    *checksum = stripe_sum(g, kStripeSum);
}

// ------------------------------------------------------------------ adjacency
// an adjacency of at most one tile: gathered and sorted in LDS by one workgroup
__global__ __launch_bounds__(kOsThreads) void k_adj_tile(GraphView g, uint32_t u, int passes,
                                                         uint32_t* out) {
    __shared__ TileSortLds lds;
    const VRec r = g.vt[u];
    uint64_t key[kOsRounds];
#pragma unroll
    for (int j = 0; j < kOsRounds; ++j) {
        const uint64_t i = (uint64_t)j * kOsThreads + threadIdx.x;
        key[j] = i < r.deg ? g.pool[slot_addr(g, r, (uint32_t)i)] : ~0ull;
    }
    tile_sort(key, r.deg, passes, ~0ull, lds);
#pragma unroll
    for (int j = 0; j < kOsRounds; ++j) {
        const uint64_t i = (uint64_t)j * kOsThreads + threadIdx.x;
        if (i < r.deg) out[i] = (uint32_t)key[j];
    }
}

// a longer one: destinations as 64-bit keys for the one-sweep sort, and back
__global__ __launch_bounds__(kThreads) void k_adj_gather64(GraphView g, uint32_t u,
                                                           uint64_t* keys) {
    const VRec r = g.vt[u];
    for (uint64_t s = tidx(); s < r.deg; s += (uint64_t)gridDim.x * kThreads)
        keys[s] = g.pool[slot_addr(g, r, (uint32_t)s)];
}

__global__ __launch_bounds__(kThreads) void k_adj_low(const uint64_t* keys, uint64_t n,
                                                      uint32_t* out) {
    const uint64_t i = tidx();
    if (i < n) out[i] = (uint32_t)keys[i];
}

void adjacency(gv_graph* g, uint32_t u, uint32_t* out, uint64_t cap, uint64_t* degree) {
    Ctx& c = g->ctx;
    const GraphView& v = g->v;
    *degree = 0;
    if ((uint64_t)u >= v.n_cap) fail(GV_ERANGE, "vertex id >= capacity");
    VRec r;
    hip_check(hipMemcpyAsync(&r, v.vt + u, sizeof(VRec), hipMemcpyDeviceToHost, c.stream),
              "hipMemcpyAsync");
    hip_check(hipStreamSynchronize(c.stream), "hipStreamSynchronize");
    *degree = r.deg;
    if (cap < r.deg) fail(GV_ERANGE, "adjacency buffer too small");
    if (r.deg == 0) return;
    if (!out) fail(GV_EINVAL, "null output");
    const uint64_t d = r.deg;
    const int bits = std::max<int>((int)v.L, 1);
    if (d <= kOsTile) {
        // one kernel: gather and sort in LDS
        c.launch("adj_sort", k_adj_tile, 1, kOsThreads, v, u, os_passes(bits), out);
        hip_check(hipStreamSynchronize(c.stream), "hipStreamSynchronize");
        return;
    }
    uint64_t *k0 = nullptr, *k1 = nullptr;
    uint32_t* state = nullptr;
    auto carve = [&](Carver& cv) {
        k0 = cv.take<uint64_t>(d);
        k1 = cv.take<uint64_t>(d);
        state = cv.take<uint32_t>(os_words(d, bits));
    };
    {
        Carver mz(nullptr);
        carve(mz);
        g->scratch.ensure(mz.used, c.stream);
        Carver cv(g->scratch.ptr);
        carve(cv);
    }
    c.launch("adj_gather", k_adj_gather64, std::min<uint64_t>(div_up(d, kThreads), 1024),
             kThreads, v, u, k0);
    const bool flip = sort_keys(g, k0, k1, d, bits, state);  // synchronous
    c.launch("adj_copy", k_adj_low, div_up(d, kThreads), kThreads,
             (const uint64_t*)(flip ? k1 : k0), d, out);
    hip_check(hipStreamSynchronize(c.stream), "hipStreamSynchronize");
}

// ------------------------------------------------------------------ audit
__global__ __launch_bounds__(kThreads) void k_zero_u32(uint32_t* a, uint64_t n) {
    const uint64_t i = tidx();
    if (i < n) a[i] = 0;
}

// one wave per vertex: owned blocks are counted, slots and records checked
__global__ __launch_bounds__(kThreads) void k_audit_vertices(GraphView g, uint32_t* seen) {
    const uint32_t lane = lane_id();
    const uint64_t nw = (uint64_t)gridDim.x * kWaves;
    const unsigned long long bump = g.ctr->bump;
    unsigned long long bad = 0;
    for (uint64_t u = gwave(); u < g.n_cap; u += nw) {
        const VRec r = g.vt[u];
        const bool act = is_active(g, u);
        if (lane == 0 && g.vlost[u] != 0u) bad++;  // vertex-delete scratch left set
        if (!act) {
            if (lane == 0 && (r.deg != 0 || r.dcls != kNoDir)) bad++;
            continue;
        }
        const uint32_t nb = nblocks(g, r.deg);
        if (r.dcls != kNoDir) {
            if (r.dcls >= kMaxClass || (1ull << r.dcls) < nb ||
                (uint64_t)r.dir + (1ull << r.dcls) > g.dir_cap) {
                if (lane == 0) bad++;
                continue;
            }
        } else if (nb > 1) {
            if (lane == 0) bad++;
            continue;
        }
        for (uint32_t j = lane; j < nb; j += 64) {
            const uint32_t id = block_of(g, r, j);
            if (id >= bump) {
                bad++;
            } else {
                atomicAdd(&seen[id], 1u);
                const uint2 ow = g.bown[id];  // the owner record names this vertex and index
                if (ow.x != (uint32_t)u || ow.y != j) bad++;
            }
        }
        for (uint32_t s = lane; s < r.deg; s += 64) {
            const uint32_t id = block_of(g, r, s >> g.log2B);
            if (id >= bump) continue;
            const uint32_t x = g.pool[((uint64_t)id << g.log2B) + (s & (g.B - 1))];
            if (x == kTomb || !is_active(g, x)) bad++;
        }
    }
    bad = wave_sum(bad);
    if (lane == 0 && bad) atomicAdd(&g.ctr->violations, bad);
}

__global__ __launch_bounds__(kThreads) void k_audit_free(GraphView g, uint32_t* seen) {
    const uint64_t i = tidx();
    if (i >= g.ctr->free_cnt) return;
    const uint32_t id = g.free_stack[i];
    if (id >= g.ctr->bump) atomicAdd(&g.ctr->violations, 1ull);
    else atomicAdd(&seen[id], 1u);
}

__global__ __launch_bounds__(kThreads) void k_audit_seen(GraphView g, const uint32_t* seen,
                                                         uint64_t n) {
    __shared__ unsigned long long lds[kWaves];
    const uint64_t i = tidx();
    unsigned long long bad = (i < n && seen[i] != 1u) ? 1ull : 0ull;
    bad = block_sum(bad, lds);
    if (threadIdx.x == 0 && bad) atomicAdd(&g.ctr->violations, bad);
}

uint64_t audit(gv_graph* g) {
    Ctx& c = g->ctx;
    const GraphView& v = g->v;
    read_counters(g);
    const uint64_t bump = g->hctr->bump;
    const uint64_t nfree = g->hctr->free_cnt;
    uint64_t bad = 0;
    if (nfree > bump || bump > v.cap_blocks) bad++;
    uint32_t* seen = nullptr;
    {
        Carver mz(nullptr);
        mz.take<uint32_t>(std::max<uint64_t>(bump, 1));
        g->scratch.ensure(mz.used, c.stream);
        Carver cv(g->scratch.ptr);
        seen = cv.take<uint32_t>(std::max<uint64_t>(bump, 1));
    }
    set_u64(g, &v.ctr->violations, 0);
    c.launch("audit_zero", k_zero_u32, div_up(std::max<uint64_t>(bump, 1), kThreads), kThreads,
             seen, bump);
    c.launch("audit_vertices", k_audit_vertices,
             std::min<uint64_t>(div_up(v.n_cap, kWaves), 4096), kThreads, v, seen);
    if (nfree)
        c.launch("audit_free", k_audit_free, div_up(nfree, kThreads), kThreads, v, seen);
    if (bump)
        c.launch("audit_seen", k_audit_seen, div_up(bump, kThreads), kThreads, v,
                 (const uint32_t*)seen, bump);
    read_counters(g);
    return bad + g->hctr->violations;
}

}  // namespace gv

namespace gv {

// ------------------------------------------------------------------ block size
// blocks the adjacencies would hold with 2^lb slots per block (low half) and
// vertices of non-zero degree (high half), one atomic per workgroup
__global__ __launch_bounds__(kThreads) void k_layout_count(GraphView g, uint32_t lb,
                                                           unsigned long long* out) {
    __shared__ unsigned long long lds[kWaves];
    const uint64_t v = tidx();
    unsigned long long blocks = 0, nz = 0;
    if (v < g.n_cap && is_active(g, v)) {
        const uint32_t d = g.vt[v].deg;
        blocks = ((uint64_t)d + (1ull << lb) - 1) >> lb;
        nz = d > 0;
    }
    blocks = block_sum(blocks, lds);
    nz = block_sum(nz, lds);
    if (threadIdx.x == 0 && (blocks | nz)) atomicAdd(out, blocks | (nz << 32));
}

// source of every dumped edge: the vertex whose CSR range holds it
__global__ __launch_bounds__(kThreads) void k_layout_src(const unsigned long long* offs,
                                                         uint64_t ncap, uint64_t m,
                                                         uint32_t* src) {
    const uint64_t i = tidx();
    if (i >= m) return;
    uint64_t lo = 0, hi = ncap;  // last v with offs[v] <= i
    while (hi - lo > 1) {
        const uint64_t mid = (lo + hi) >> 1;
        if (offs[mid] <= i) lo = mid;
        else hi = mid;
    }
    src[i] = (uint32_t)lo;
}

namespace {

// (blocks with 2^lb slots, vertices of non-zero degree)
std::pair<uint64_t, uint64_t> layout_count(gv_graph* g, uint32_t lb) {
    const GraphView& v = g->v;
    set_u64(g, &v.ctr->checksum, 0);
    g->ctx.launch("relayout", k_layout_count, div_up(v.n_cap, kThreads), kThreads, v, lb,
                  &v.ctr->checksum);
    read_counters(g);
    const unsigned long long x = g->hctr->checksum;
    return {x & 0xffffffffull, x >> 32};
}

struct DevBuf {
    void* p = nullptr;
    ~DevBuf() {
        if (p) hipFree(p);
    }
    template <typename T>
    T* get(size_t count) {
        hip_check(dev_alloc(&p, std::max<size_t>(count * sizeof(T), 8)), "hipMalloc relayout");
        return (T*)p;
    }
};

}  // namespace

uint32_t adapted_block_slots(gv_graph* g) {
    read_counters(g);
    const uint64_t edges = g->hctr->live_edges;
    const uint64_t nonzero = layout_count(g, 0).second;
    return paper_block_rule(edges, nonzero);
}

// The same edges (and attribute words) in blocks of block_slots slots: dump,
// rebuild with the pool's byte budget, restore the activity bitmap, write the
// words back.  Checks first that the new layout fits, so that a graph that
// would not fit stays as it is (GV_ENOMEM).
void relayout(gv_graph* g, uint32_t block_slots) {
    Ctx& c = g->ctx;
    GraphView& v = g->v;
    if (block_slots == v.B) return;
    read_counters(g);
    // a rebuild clears the error words: report a pending one first
    if (g->hctr->err_sticky) fail((int)g->hctr->err_sticky, "an earlier batch failed");
    const uint64_t m = g->hctr->live_edges;
    if (m >= kOsMaxKeys) fail(GV_EINVAL, "2^30 or more edges");
    const uint64_t budget = v.cap_blocks * v.B * 4ull;
    const uint64_t cap_new = std::min<uint64_t>(budget / (4ull * block_slots), 0xfffffff0ull);
    if (layout_count(g, log2_exact(block_slots)).first > cap_new)
        fail(GV_ENOMEM, "the graph does not fit the pool with that block size");
    const uint64_t words = (v.n_cap + 31) / 32;
    DevBuf b_offs, b_dst, b_src, b_attr, b_found, b_act;
    auto* offs = b_offs.get<uint64_t>(v.n_cap + 1);
    auto* dst = b_dst.get<uint32_t>(m);
    auto* src = b_src.get<uint32_t>(m);
    auto* act = b_act.get<uint32_t>(words);
    uint32_t* attr = v.A ? b_attr.get<uint32_t>(m * v.A) : nullptr;
    uint64_t ck = 0, e = 0;
    dump(g, offs, dst, m, &ck, &e);
    if (e != m) fail(GV_EDEVICE, "edge count changed during a relayout");
    if (m)
        c.launch("relayout", k_layout_src, div_up(m, kThreads), kThreads,
                 (const unsigned long long*)offs, (uint64_t)v.n_cap, m, src);
    if (attr && m) edge_attrs(g, src, dst, m, b_found.get<uint8_t>(m), attr, nullptr);
    hip_check(hipMemcpyAsync(act, v.active, words * 4, hipMemcpyDeviceToDevice, c.stream),
              "hipMemcpyAsync");
    hip_check(hipStreamSynchronize(c.stream), "hipStreamSynchronize");
    // from here the old layout is gone: a failure leaves the graph unusable
    g->dead = true;
    dev_free(g->mem_pool, true);  // (the stream was waited for)
    g->mem_pool = nullptr;
    gv_config cfg{};
    cfg.block_slots = block_slots;
    cfg.pool_bytes = budget;
    cfg.vertex_capacity = v.n_cap;
    cfg.edge_attr_words = v.A;
    bulk_build(g, v.n_cap, src, dst, m, cfg);
    hip_check(hipMemcpyAsync(v.active, act, words * 4, hipMemcpyDeviceToDevice, c.stream),
              "hipMemcpyAsync");
    if (attr && m) edge_attrs(g, src, dst, m, nullptr, nullptr, attr);
    hip_check(hipStreamSynchronize(c.stream), "hipStreamSynchronize");
    g->dead = false;
    ++g->table_gen;  // recorded plans hold the old layout
}

}  // namespace gv
