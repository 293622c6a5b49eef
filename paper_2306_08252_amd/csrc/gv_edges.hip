// gv_edges.hip -- batched edge insert, delete and query.
//
// One pipeline serves the three operations (GraphVine Sec. 4.5-4.6, Alg. 1-3,
// re-designed for wave64):
//   pack +    every pair is checked against the activity bitmap and becomes the
//   sort      key (src << L) | dst; an invalid pair gets a key past every valid
//             one.  Up to kRankMax pairs one kernel packs and sorts by rank;
//             larger batches are packed with the digit counts and go through
//             the onesweep LSD radix sort (queries compact their valid pairs
//             with their input positions first).  The batch is then grouped by
//             source and ordered by destination inside each source segment
//             (the paper's host CSR conversion, Sec. 4.3).
//   segments  one kernel over tiles of the sorted keys: segment heads give the
//             touched sources T (a 32-byte record each: segment, vertex record)
//             and repeated pairs; each touched adjacency is cut into work
//             items of `chunk` slots.  A tile takes its sources' and items'
//             places with one atomic each, so T is in tile order only inside a
//             tile, and no scan over the batch is needed.
//   probe     sources with few slots and a short segment by four lanes each
//             (slots and segment loaded whole, all pairs compared); the others
//             by a wave per work item that stages the segment's destinations
//             in LDS and binary-searches each slot value there, with the loads
//             of its next three items in flight.
//             Insert: mark batch entries that already exist (set semantics).
//             Delete: mark hits, remember their slot.
//             Query:  mark every query equal to a stored edge.
//   plan      insert and delete, the same tiles: each source's kept pairs
//             (neither repeated nor present) or hits, block demand or freed
//             blocks, directory growth; the tile's share is placed with one
//             atomic.  The last tile to finish runs the one-wave plan: an
//             insert checks capacity before any state is written
//             (all-or-nothing; blocks come from the free-list top first, then
//             the bump pointer: the prefix-sum pop of Sec. 4.5.1).
//   insert:   commit: kept pairs to slots deg + rank, new block ids,
//             directory moves and vertex records; old directory segments freed.
//   delete:   per-source compaction pairs the holes below the new degree with
//             the survivors above it, by rank (one launch: a workgroup per
//             hub first, then lanes and waves for the other sources); emptied
//             blocks are pushed on the free list at planned positions
//             (reclamation, Sec. 4.2).
//   query:    answers are scattered back to input order.
#include <algorithm>
#include <cstddef>
#include <type_traits>

#include "gv_graph.h"
#include "gv_prim.h"

namespace gv {

constexpr int kStageLog = 7;                   // log2(kStage)
constexpr int kStage = 1 << kStageLog;         // segment entries staged in LDS
#ifndef GV_BIG_R
#define GV_BIG_R 256
#endif
#ifndef GV_LANE_SEG
#define GV_LANE_SEG 16
#endif
#ifndef GV_LANE_R
#define GV_LANE_R 8
#endif
constexpr int kProbeWaves = 8;                  // waves per SIMD of the probe
constexpr uint32_t kBigR = GV_BIG_R;           // deletes per source handled by a workgroup
constexpr uint32_t kBigGroups = 256;           // workgroups for those sources
constexpr uint32_t kLaneCopy = 8;              // directory entries a lane copies or adds
constexpr uint32_t kLaneSeg = GV_LANE_SEG;     // segment entries a lane compacts
constexpr uint32_t kLaneR = GV_LANE_R;         // hits a lane compacts
constexpr uint32_t kNoHit = 0xFFFFFFFFu;       // hit position of a pair not found (delete)
constexpr uint32_t kHeavy = 0x100u;            // flag bit in t_dreq: whole waves grow this source
constexpr uint32_t kClassMask = 0xFFu;         // t_dreq & kClassMask: requested class or kNoDir

// probe mode of the attribute calls: a query that also records the slot of
// every occurrence it finds
constexpr int kLocate = 3;

// Counters of one batch, in the batch's own buffer (with the sort overlap on,
// a batch's packing clears them while the batch before it still uses its
// own), cleared by its first kernel.  Every word that a kernel adds to from
// all of its workgroups and then uses is a word of its own that each
// workgroup touches once.
struct alignas(128) BatchCtr {
    unsigned long long n_valid, key_sum;  // valid pairs, and the mix64 sum of their keys
    uint32_t n_big, n_heavy;              // sources left to workgroups / to whole waves
    uint32_t nohash;                      // keys arrived sorted: no multiset check
    uint32_t sort_err;                    // a wait of the batch's own sort ran out
    unsigned long long pad1[12];
    // touched sources (high) and work items (low: at most one per pair and one
    // per 64 slots of the pool) placed
    unsigned long long alloc;
    unsigned long long pad2[15];
    // insert: blocks needed (low), directory segments given back (high);
    // delete: blocks freed (low), sources for whole waves (high)
    unsigned long long demand;
    unsigned long long pad3[15];
    unsigned long long done;  // tiles planned (high); their pairs kept or hits (low)
    unsigned long long pad4[15];
    unsigned long long stripe[64][16];    // kStripe* sums, a line each
};
enum { kStripeHash = 0, kStripeUniq = 1, kStripeBlocks = 2 };

// self-contained work item: slots [s0, s1) of a source, batch segment [lo, hi);
// block j is directory entry dir + j, or (inl) dir is the only block
struct alignas(8) Item {
    uint32_t s0, s1, lo, hi;
    uint32_t dir, inl;
};

// A touched source: its batch segment [lo, hi), its vertex record as it was
// before the batch, then (plan) its kept pairs or hits r and the first of its
// blocks, needed or freed, among those of the tile that holds lo.
struct alignas(16) Src {
    uint32_t lo, hi, r, v;
    uint32_t deg, dir, dcls, need;
};

// Tiles of sorted positions: the segments, plan and commit kernels of a batch
// take one workgroup per tile of 2^tl positions.
constexpr uint32_t kTileLogMin = 6, kTileLogMax = 12;
constexpr uint32_t kTileMax = 1u << kTileLogMax;
constexpr uint32_t kTileRows = 4;  // positions per thread, at most

// attribute call of a query batch: get (out) or set (in), n * A words
struct AttrOp {
    uint32_t* out;
    const uint32_t* in;
};

struct BatchArrays {
    BatchCtr* bc;
    uint64_t* keys0;
    uint64_t* keys1;
    uint32_t* vals0;
    uint32_t* vals1;
    uint8_t* mark;
    uint32_t* hitpos;   // delete, attribute calls: slot index of each hit
    uint32_t* holes;    // delete: hole slots per segment
    Src* srcs;          // touched sources
    uint2* tiles;       // per tile: its first source, its sources
    uint2* carry;       // insert, per tile: the source whose segment runs into
                        // the tile, and that source's kept pairs before it
    uint32_t* tbase;    // per tile: first of its blocks among the batch's
    uint32_t* tkept;    // per tile inside a segment: its kept pairs or hits, plus
                        // one, once the plan has counted them (0 before)
    uint32_t* t_dreq;   // insert: requested directory class or kNoDir
    uint32_t* t_drank;  // insert: rank among requests of that class
    uint32_t* t_dold;   // insert: replaced directory segment offset
    uint32_t* t_doldc;  // insert: replaced directory segment class or kNoDir
    uint32_t* rel;      // insert: sources that give back a directory segment
    uint32_t* big;      // delete: sources with more than kBigR hits
    uint32_t* heavy;    // sources left to whole waves
    Item* items;        // work items
    unsigned long long* part;  // scan partials (query)
    uint32_t* state;    // zeroed look-back state of the sort
    uint64_t state_words;
    uint32_t* vpart;    // insert / delete: valid pairs per packing workgroup
    unsigned long long* hpart;  // insert / delete: mix64 sum of valid keys per packing workgroup
};

// log2 of the positions per tile for a batch of n pairs: about 512 tiles, so
// that two workgroups per compute unit share the work, between one wave's
// width (smaller tiles would only add workgroups) and the LDS arrays' size.
static uint32_t tile_log(uint64_t n) {
    uint32_t tl = kTileLogMin;
    while (tl < kTileLogMax && (n >> tl) > 512) ++tl;
    return tl;
}

static void carve_batch(Carver& cv, BatchArrays& A, uint64_t n, uint64_t icap, EdgeMode mode,
                        int bits) {
    A = BatchArrays{};
    const uint64_t nt = div_up(n, 1ull << tile_log(n));
    A.bc = cv.take<BatchCtr>(1);
    A.keys0 = cv.take<uint64_t>(n);
    A.keys1 = cv.take<uint64_t>(n);
    if (mode == kQuery) {
        A.vals0 = cv.take<uint32_t>(n);
        A.vals1 = cv.take<uint32_t>(n);
        A.part = cv.take<unsigned long long>(scan2_parts(n));
    }
    A.mark = cv.take<uint8_t>(n);
    // (whole groups of four; query: attribute calls)
    if (mode != kInsert) A.hitpos = cv.take<uint32_t>((n + 3) & ~3ull);
    if (mode == kDelete) {
        A.holes = cv.take<uint32_t>(n);
        A.big = cv.take<uint32_t>(n);
    }
    if (mode != kQuery) {
        A.heavy = cv.take<uint32_t>(n);
        A.tbase = cv.take<uint32_t>(nt);
    }
    A.srcs = cv.take<Src>(n);
    A.tiles = cv.take<uint2>(nt);
    if (mode == kInsert) {
        A.carry = cv.take<uint2>(nt);
        A.t_dreq = cv.take<uint32_t>(n);
        A.t_drank = cv.take<uint32_t>(n);
        A.t_dold = cv.take<uint32_t>(n);
        A.t_doldc = cv.take<uint32_t>(n);
        A.rel = cv.take<uint32_t>(n);
    }
    A.items = cv.take<Item>(icap);
    A.state_words = os_zero_words(n, bits, mode == kQuery);  // the part the batch zeroes
    A.state = cv.take<uint32_t>(os_words(n, bits, mode == kQuery));
    A.vpart = cv.take<uint32_t>(kHistGroups);
    A.hpart = cv.take<unsigned long long>(kHistGroups);
    if (mode != kQuery) A.tkept = cv.take<uint32_t>(nt);
}

__device__ __forceinline__ uint64_t thread_index() {
    return (uint64_t)blockIdx.x * kThreads + threadIdx.x;
}

// ------------------------------------------------------------------ begin
// Clears the batch's counters; called by one whole workgroup of nt threads.
__device__ __forceinline__ void clear_batch(BatchCtr* bc, uint32_t t, uint32_t nt) {
    uint32_t* w = (uint32_t*)bc;
    for (uint32_t i = t; i < sizeof(BatchCtr) / 4; i += nt) w[i] = 0u;
}

__global__ __launch_bounds__(kThreads) void k_begin(BatchCtr* bc) {
    clear_batch(bc, threadIdx.x, kThreads);
}

// ------------------------------------------------------------------ pack
// Scan sources follow the gather interface of scan2: load() performs every
// memory read of an element at addresses that are valid whether or not the
// element is live, value() and the sinks only compute and store.
struct PackIn {
    GraphView g;
    const uint32_t* src;
    const uint32_t* dst;
    struct Rec {
        uint32_t s, d;
        bool ok;
    };
    __device__ uint64_t limit(uint64_t n) const { return n; }
    __device__ Rec load(uint64_t i, bool) const { return Rec{src[i], dst[i], false}; }
    __device__ void deref(Rec& r) const { r.ok = active_bit(g, r.s) & active_bit(g, r.d); }
    __device__ unsigned long long value(uint64_t, const Rec& r) const { return r.ok ? 1ull : 0ull; }
};

struct PackOut {
    uint32_t L;
    uint64_t* keys;
    uint32_t* vals;     // queries: input position of each valid key
    uint8_t* answer;    // queries: invalid pairs are answered here
    __device__ void operator()(uint64_t i, const PackIn::Rec& r, uint64_t,
                               unsigned long long pos) const {
        if (r.ok) {
            keys[pos] = ((uint64_t)r.s << L) | r.d;
            if (vals) vals[pos] = (uint32_t)i;
        } else if (answer) {
            answer[i] = 0;
        }
    }
};

// Insert and delete batches: pack without compaction.  Every pair keeps its
// input position; a pair with an inactive or out-of-range endpoint gets the
// all-ones key of the sort's bit width, which sorts after every valid key.
// All such keys are equal, so whether or not a valid pair shares that key,
// the first n_valid sorted keys are exactly the valid ones.  The same kernel
// clears the batch's look-back state and counters and counts the sort's
// digits (per workgroup, summed by the next kernel together with the valid
// pairs).
__global__ __launch_bounds__(kOsThreads) void k_pack_hist(GraphView g, const uint32_t* src,
                                                          const uint32_t* dst, uint64_t n,
                                                          int passes, uint64_t sentinel,
                                                          uint64_t* keys, BatchCtr* bc,
                                                          uint32_t* state, uint64_t zero_words,
                                                          uint32_t* hpart, uint32_t* vpart,
                                                          unsigned long long* kpart) {
    __shared__ uint32_t h[kOsHistCopies][8][kRadix];
    __shared__ uint32_t s_v[kOsWaves];
    __shared__ unsigned long long s_k[kOsWaves];
    const uint32_t t = threadIdx.x;
    for (uint64_t i = (uint64_t)blockIdx.x * kOsThreads + t; i < zero_words;
         i += (uint64_t)gridDim.x * kOsThreads)
        state[i] = 0;
    if (blockIdx.x == 0) clear_batch(bc, t, kOsThreads);
    for (int i = t; i < kOsHistCopies * 8 * kRadix; i += kOsThreads) (&h[0][0][0])[i] = 0;
    __syncthreads();
    const uint32_t copy = kOsHistCopies == 1 ? 0u : (t >> 6) & (kOsHistCopies - 1);
    uint32_t valid = 0;
    unsigned long long khash = 0;  // multiset hash of the valid keys (checked after the sort)
    const uint64_t ntiles = (n + kHistTile - 1) / kHistTile;
    for (uint64_t tl = blockIdx.x; tl < ntiles; tl += gridDim.x) {
        const uint64_t i = tl * kHistTile + t;
        if (i >= n) continue;
        const uint32_t su = src[i], du = dst[i];
        const bool ok = active_bit(g, su) & active_bit(g, du);
        const uint64_t key = ok ? ((uint64_t)su << g.L) | du : sentinel;
        keys[i] = key;
        valid += ok ? 1u : 0u;
        khash += ok ? mix64(key) : 0ull;
        for (int p = 0; p < passes; ++p)
            atomicAdd(&h[copy][p][(uint32_t)(key >> (p * kRadixBits)) & (kRadix - 1)], 1u);
    }
    const uint32_t vw = (uint32_t)wave_sum((unsigned long long)valid);
    const unsigned long long kw = wave_sum(khash);
    if (lane_id() == 0) {
        s_v[t >> 6] = vw;
        s_k[t >> 6] = kw;
    }
    __syncthreads();
    uint32_t* out = hpart + (uint64_t)blockIdx.x * passes * kRadix;
    for (int i = t; i < passes * kRadix; i += kOsThreads) {
        uint32_t x = 0;
#pragma unroll
        for (int c = 0; c < kOsHistCopies; ++c) x += h[c][i / kRadix][i % kRadix];
        out[i] = x;
    }
    if (t == 0) {
        uint32_t x = 0;
        unsigned long long y = 0;
        for (int w = 0; w < kOsWaves; ++w) {
            x += s_v[w];
            y += s_k[w];
        }
        vpart[blockIdx.x] = x;
        kpart[blockIdx.x] = y;
    }
}

// Batches of at most kRankMax pairs: packed and sorted by rank (gv_prim.h).
struct EdgeKeys {
    static constexpr bool kGathers = true;
    GraphView g;
    const uint32_t* src;
    const uint32_t* dst;
    uint8_t* answer;  // queries: invalid pairs are answered here
    BatchCtr* bc;
    struct Raw {
        uint32_t s, d;
    };
    __device__ Raw raw(uint64_t i) const { return Raw{src[i], dst[i]}; }
    __device__ uint64_t key(const Raw& r) const {
        const bool ok = active_bit(g, r.s) & active_bit(g, r.d);
        return ok ? ((uint64_t)r.s << g.L) | r.d : 1ull << (2 * g.L);
    }
    __device__ void own(uint64_t i, uint64_t key) const {
        if (answer && (key >> (2 * g.L))) answer[i] = 0;
    }
    // by the first workgroup, which sees every key
    __device__ void begin(uint32_t t, uint32_t nt) const { clear_batch(bc, t, nt); }
    __device__ bool counted(uint64_t key) const { return (key >> (2 * g.L)) == 0; }
    __device__ void totals(unsigned long long n, unsigned long long sum) const {
        bc->n_valid = n;
        bc->key_sum = sum;
    }
};

// ------------------------------------------------------------------ segments
// Small items: a source with at most kSmallLanes * kSmallDeg slots and at
// most kSmallSeg pairs in its batch segment is probed by kSmallLanes lanes,
// kSmallDeg slots each, from its source record; it has no work items.
constexpr uint32_t kSmallDeg = 16;    // slots per lane (whole 16-byte groups of a block)
constexpr uint32_t kSmallLanes = 4;   // lanes per small item
#ifndef GV_SMALL_SEG
#define GV_SMALL_SEG 8
#endif
constexpr uint32_t kSmallSeg = GV_SMALL_SEG;
__device__ __forceinline__ bool small_item(uint32_t B, uint32_t deg, uint32_t len) {
    return B >= 4 && deg > 0 && deg <= kSmallLanes * kSmallDeg && len <= kSmallSeg;
}

// Valid pairs of the batch: none after a look-back wait ran out (the keys are
// not sorted).  Every kernel of a batch has to decide alike in all of its
// workgroups, and alike with the kernels after it: a tile planned as failed has
// no block places for the commit.  So nothing that runs beside the batch writes
// what it reads: a sort, which may be that of a later batch on the side stream,
// flags its own batch's counters only, and the batch's first kernel on the
// graph's stream carries the flag over to the graph's.
__device__ __forceinline__ uint64_t batch_pairs(const DevCounters* c, const BatchCtr* bc,
                                                uint64_t n) {
    return (c->err_wait | bc->sort_err) ? 0ull : min((uint64_t)bc->n_valid, n);
}

// First position in keys[lo, hi) whose key is at least x, by one wave: 64
// probes a step.
__device__ __forceinline__ uint64_t wave_lower_bound(const uint64_t* keys, uint64_t lo,
                                                     uint64_t hi, uint64_t x) {
    const uint32_t lane = lane_id();
    while (lo < hi) {
        const uint64_t step = (hi - lo + 63) / 64;
        const uint64_t p = lo + lane * step;
        const uint64_t less = ballot(p < hi && keys[p] < x);
        if (!less) return lo;
        const uint64_t k = popc64(less);  // (the keys are in order)
        lo += (k - 1) * step + 1;
        hi = min(hi, lo - 1 + step);
    }
    return lo;
}

// Exclusive ranks of a flag over a tile's positions (row j of thread t is
// position j * T + t), by ballots: one LDS exchange of the per-wave counts.
// Returns the number of set flags; cnt holds kTileRows * T / 64 words.
template <int T, uint32_t R>
__device__ __forceinline__ uint32_t tile_ranks(const bool (&f)[R], uint32_t (&rank)[R],
                                               uint32_t* cnt) {
    constexpr uint32_t W = T / 64, N = R * W;
    static_assert(N <= 64, "one wave scans the counts");
    const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint64_t m[R];
#pragma unroll
    for (uint32_t j = 0; j < R; ++j) {
        m[j] = ballot(f[j]);
        if (lane_id() == 0) cnt[j * W + w] = popc64(m[j]);
    }
    __syncthreads();
    const uint32_t c = lane_id() < N ? cnt[lane_id()] : 0u;
    const uint32_t inc = wave_incl_scan(c);  // every wave for itself
#pragma unroll
    for (uint32_t j = 0; j < R; ++j)
        rank[j] = wave_read(inc - c, j * W + w) + rank_below(m[j]);
    const uint32_t total = wave_read(inc, 63);
    __syncthreads();
    return total;
}

// The same for counts: exclusive sums in position order, and their total.
template <int T, typename V, uint32_t R>
__device__ __forceinline__ V tile_sums(const V (&x)[R], V (&ex)[R], V* cnt) {
    constexpr uint32_t W = T / 64, N = R * W;
    static_assert(N <= 64, "one wave scans the sums");
    const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
    for (uint32_t j = 0; j < R; ++j) {
        const V inc = wave_incl_scan(x[j]);
        if (lane_id() == 63) cnt[j * W + w] = inc;
        ex[j] = inc - x[j];
    }
    __syncthreads();
    if constexpr (R == 1) {  // few: every thread adds them up
        V before = 0, all = 0;
#pragma unroll
        for (uint32_t i = 0; i < W; ++i) {
            const V v = cnt[i];
            before += i < w ? v : V(0);
            all += v;
        }
        ex[0] += before;
        return all;
    }
    const V c = lane_id() < N ? cnt[lane_id()] : V(0);
    const V inc = wave_incl_scan(c);
#pragma unroll
    for (uint32_t j = 0; j < R; ++j) ex[j] += wave_read(inc - c, j * W + w);
    return wave_read(inc, 63);
}

// Segments, sources and work items of a tile of the sorted keys.  Also writes
// the marks (dup_mark: 1 on a repeated pair, which an insert does not keep)
// and a delete's hit positions (none yet), checks the sort (every key at least
// its predecessor, else err_order = 2; the mix64 sum of the sorted keys goes to
// the hash stripes, which the probe compares with the packed keys' sum) and
// counts distinct pairs and blocks.
//
// A segment that runs past the tile belongs to the tile of its head, which
// finds its end by a wave-wide search.  Every position reads its source's
// vertex record with its key, before it is known to be a head, and both before
// the batch's counters have arrived (at positions clamped to the buffers).
// Work items are written by all the threads of the workgroup, each finding its
// item's source among the tile's (a hub's items spread over the workgroup;
// written by its own lane or wave they took up to 1.7 times as long).
//
// Bound: latency, keys -> records -> the tile's places -> the sources: 10^3
// pairs 10.2 -> 6.6 us, 10^4 pairs 10.0 -> 6.3, 10^6 pairs 25.5 -> 15.6, 10^7
// pairs 99 -> 62 (R-MAT 2^20 / 2^24, the last 2^22 / 2^26) against records read
// by the heads alone, after the counters and the keys.  The two scans over the
// batch that it replaced (their reduce and apply kernels, a middle one past
// 2^21 pairs, and 32 bytes written per source for its small item) took 21.8 us
// for 10^4 pairs, 33.3 and 218.
template <int T, uint32_t R>
__global__ __launch_bounds__(T, 8) void k_segments(GraphView g, const uint64_t* keys, uint64_t n,
                                                BatchCtr* bc, uint32_t tl, uint8_t* mark,
                                                int dup_mark, uint32_t* hitpos, Src* srcs,
                                                uint2* tiles, uint32_t* tkept, Item* items,
                                                uint64_t icap, uint32_t chunk) {
    constexpr uint32_t kTile = T * R;
    // the tile's sources: position (and whether `dir` is the only block),
    // degree, directory, first work item
    __shared__ uint32_t s_pos[kTile], s_deg[kTile], s_dir[kTile], s_base[kTile];
    constexpr uint32_t kInl = 1u << 31;
    __shared__ uint32_t s_cnt[R * T / 64], s_cnt2[R * T / 64];
    __shared__ unsigned long long s_sum[3], s_at;
    __shared__ uint32_t s_end;
    const uint32_t t = threadIdx.x, lane = lane_id();
    const uint64_t p0 = (uint64_t)blockIdx.x << tl;
    const uint32_t L = g.L;
    const uint32_t tile = 1u << tl;
    uint64_t k[R], q[R];
#pragma unroll
    for (uint32_t j = 0; j < R; ++j) {
        const uint64_t i = min(p0 + min(j * T + t, tile - 1), n - 1);
        k[j] = keys[i];
        q[j] = keys[i ? i - 1 : 0];
    }
    const uint64_t ka = keys[min(p0 + tile, n) - 1], kb = keys[min(p0 + tile, n - 1)];
    const uint64_t lim = batch_pairs(g.ctr, bc, n);
    if (blockIdx.x == 0 && t == 0 && bc->sort_err) g.ctr->err_wait = 1u;
    // a valid key's source is below n_cap already; the bound keeps even a
    // corrupted key's record read inside the table
    VRec rec[R];
#pragma unroll
    for (uint32_t j = 0; j < R; ++j)
        rec[j] = g.vt[min((uint32_t)(k[j] >> L) & (uint32_t)((1ull << L) - 1),
                           (uint32_t)(g.n_cap - 1))];
    if (p0 >= lim) {
        if (t == 0) tiles[blockIdx.x] = make_uint2(0u, 0u);
        return;
    }
    const uint32_t np = (uint32_t)min((uint64_t)tile, lim - p0);
    if (t < 3) s_sum[t] = 0ull;
    bool head[R];
    unsigned long long hash = 0, uniq = 0;
    bool bad = false;
#pragma unroll
    for (uint32_t j = 0; j < R; ++j) {
        const uint32_t p = j * T + t;
        const bool in = p < np, first = p0 + p == 0;
        head[j] = in && (first || (k[j] >> L) != (q[j] >> L));
        const bool un = in && (first || k[j] != q[j]);
        uniq += un;
        bad |= in && !first && k[j] < q[j];
        hash += in ? mix64(k[j]) : 0ull;
        if (in) mark[p0 + p] = (dup_mark && !un) ? 1 : 0;
        if (in && hitpos) hitpos[p0 + p] = kNoHit;
    }
    if (bad) g.ctr->err_order = 2;
    uint32_t rank[R];
    const uint32_t nh = tile_ranks<T>(head, rank, s_cnt);
#pragma unroll
    for (uint32_t j = 0; j < R; ++j)
        if (head[j]) {
            s_pos[rank[j]] = j * T + t | (rec[j].dcls == kNoDir ? kInl : 0u);
            s_deg[rank[j]] = rec[j].deg;
            s_dir[rank[j]] = rec[j].dir;
        }
    if (t >= T - 64) {
        // the end of the segment that holds the tile's last key
        const uint64_t pe = p0 + np;
        uint64_t end = pe;
        if (pe < lim && (ka >> L) == (kb >> L))  // (then the tile is full)
            end = wave_lower_bound(keys, pe, lim, ((ka >> L) + 1) << L);
        if (lane == 0) s_end = (uint32_t)end;
    }
    __syncthreads();
    uint32_t cnt[R], ex[R], end[R];
    unsigned long long blocks = 0;
#pragma unroll
    for (uint32_t j = 0; j < R; ++j) {
        cnt[j] = end[j] = 0;
        if (!head[j]) continue;
        end[j] = rank[j] + 1 < nh ? (uint32_t)p0 + (s_pos[rank[j] + 1] & ~kInl) : s_end;
        blocks += nblocks(g, rec[j].deg);
        if (!small_item(g.B, rec[j].deg, end[j] - ((uint32_t)p0 + j * T + t)))
            cnt[j] = (rec[j].deg + chunk - 1) / chunk;
    }
    const uint32_t ni = tile_sums<T>(cnt, ex, s_cnt2);
#pragma unroll
    for (uint32_t j = 0; j < R; ++j)
        if (head[j]) s_base[rank[j]] = ex[j];
    if (t == 0) {
        s_at = nh ? atomicAdd(&bc->alloc, (unsigned long long)nh << 32 | ni) : 0ull;
        tiles[blockIdx.x] = make_uint2((uint32_t)(s_at >> 32), nh);
        if (!nh && tkept) tkept[blockIdx.x] = 0u;
    }
    hash = wave_sum(hash);
    uniq = wave_sum(uniq);
    blocks = wave_sum(blocks);
    if (lane == 0) {
        atomicAdd(&s_sum[0], hash);
        atomicAdd(&s_sum[1], uniq);
        atomicAdd(&s_sum[2], blocks);
    }
    __syncthreads();
    if (t < 3) atomicAdd(&bc->stripe[blockIdx.x & 63][t], s_sum[t]);
    const uint32_t t0 = (uint32_t)(s_at >> 32), i0 = (uint32_t)s_at;
#pragma unroll
    for (uint32_t j = 0; j < R; ++j) {
        if (!head[j]) continue;
        Src x;
        x.lo = (uint32_t)p0 + j * T + t;
        x.hi = end[j];
        x.r = 0;
        x.v = (uint32_t)(k[j] >> L) & (uint32_t)((1ull << L) - 1);
        x.deg = rec[j].deg;
        x.dir = rec[j].dir;
        x.dcls = rec[j].dcls;
        x.need = 0;
        srcs[t0 + rank[j]] = x;
    }
    for (uint32_t m = t; m < ni; m += T) {
        // the last source whose items start at or before m
        uint32_t lo = 0, hi = nh;
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if (s_base[mid] <= m) lo = mid;
            else hi = mid;
        }
        const uint32_t a = s_pos[lo];
        Item it;
        it.s0 = (m - s_base[lo]) * chunk;
        it.s1 = min(s_deg[lo], it.s0 + chunk);
        it.lo = (uint32_t)p0 + (a & ~kInl);
        it.hi = lo + 1 < nh ? (uint32_t)p0 + (s_pos[lo + 1] & ~kInl) : s_end;
        it.dir = s_dir[lo];
        it.inl = (a & kInl) != 0;
        if ((uint64_t)i0 + m < icap) items[(uint64_t)i0 + m] = it;
    }
}

// ------------------------------------------------------------------ probe
// what a stored slot si with the destination of segment position pos does;
// dup: the next position holds that destination too (queries; it is read with
// the position's own, so that the usual hit waits for nothing), and same(j)
// says so of position j
template <int MODE, typename F>
__device__ __forceinline__ void probe_hit(uint32_t lo, uint32_t len, uint32_t pos, uint32_t si,
                                          bool dup, uint8_t* mark, uint32_t* hitpos, F&& same) {
    mark[lo + pos] = 1;
    if (MODE == kDelete || MODE == kLocate) hitpos[lo + pos] = si;
    if ((MODE == kQuery || MODE == kLocate) && dup) {
        for (uint32_t j = pos + 1; j < len && same(j); ++j) {
            mark[lo + j] = 1;
            if (MODE == kLocate) hitpos[lo + j] = si;
        }
    }
}

// The U slots x of a lane, at s, s + 1, ... (one per SLOTS apart) of an item
// that ends at s1, against the batch segment [lo, lo + len), whose entries (or
// every 2^shift-th of them) are the first ns words at byte base of the LDS
// array, padded with 0xFFFFFFFF up to 2^steps - 1 (at least one pad entry, so
// that the rank can reach ns).  Searches of the slots run in lockstep, so that
// each step issues U independent reads and waits once.  Everything but x and s
// is the same for the whole wave.
template <int MODE, int U, int APART>
__device__ __forceinline__ void probe_search(const uint32_t (&x)[U], uint32_t s, uint32_t s1,
                                             uint32_t lo, uint32_t len, const char* lds,
                                             uint32_t base, uint32_t steps, uint32_t shift,
                                             const uint32_t* klo, uint32_t dmask, uint8_t* mark,
                                             uint32_t* hitpos) {
    // ranks as byte offsets into the LDS array, so that a step's read takes no
    // address arithmetic
    auto at = [&](uint32_t o) { return *(const uint32_t*)(lds + o); };
    uint32_t r[U];
#pragma unroll
    for (int u = 0; u < U; ++u) r[u] = base;
#pragma unroll
    for (int k = kStageLog - 1; k >= 0; --k) {
        if ((uint32_t)k >= steps) continue;
        const uint32_t half = 4u << k;
        uint32_t sv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) sv[u] = at(r[u] + half - 4);
#pragma unroll
        for (int u = 0; u < U; ++u) r[u] += sv[u] < x[u] ? half : 0u;
    }
    if (shift == 0) {
        const uint32_t end = base + 4 * len;
        uint32_t v[U], w[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            v[u] = at(r[u]);  // the rank is at most len < kStage
            w[u] = MODE == kQuery || MODE == kLocate ? at(r[u] + 4) : 0u;
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (v[u] == x[u] && r[u] < end && s + u * APART < s1)
                probe_hit<MODE>(lo, len, (r[u] - base) / 4, s + u * APART, w[u] == x[u], mark,
                                hitpos, [&](uint32_t j) { return at(base + 4 * j) == x[u]; });
        return;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) r[u] = (r[u] - base) / 4;
    // first segment position whose value is >= x: it lies in
    // ((r - 1) * stride, r * stride], a window of fewer than 2^shift entries
    // before the sample at r * stride (or the end of the segment); branch-free
    // lower bound in `shift` steps
    uint32_t p[U], end[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        p[u] = r[u] ? ((r[u] - 1) << shift) + 1 : 0;
        end[u] = min(r[u] << shift, len);
    }
    for (uint32_t k = shift; k-- > 0;) {
        const uint32_t half = 1u << k;
        uint32_t kv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) kv[u] = klo[2ull * min(p[u] + half - 1, len - 1)] & dmask;
#pragma unroll
        for (int u = 0; u < U; ++u)
            p[u] += (p[u] + half - 1 < end[u] && kv[u] < x[u]) ? half : 0u;
    }
    uint32_t kv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) kv[u] = klo[2ull * min(p[u], len - 1)] & dmask;
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (kv[u] == x[u] && p[u] < len && s + u * APART < s1)
            probe_hit<MODE>(lo, len, p[u], s + u * APART, true, mark, hitpos,
                            [&](uint32_t j) { return (klo[2ull * j] & dmask) == x[u]; });
}

// value of lane I of each group of four lanes
template <int I>
__device__ __forceinline__ uint32_t quad_get(uint32_t x) {
    return __builtin_amdgcn_update_dpp(0u, x, I * 0x55, 0xf, 0xf, true);
}

// The four lanes of a small item probe its adjacency in rounds of 16 slots,
// four each, against the segment's destinations (two loaded per lane,
// exchanged), all pairs compared; a round that no source of the wave has is
// skipped (most have one: the sources of a batch hold ten slots on average).
// Same marks as the search: insert and delete mark the first occurrence of a
// stored pair (delete also records the slot), query marks every occurrence.  A
// stored pair sits in one slot, so one lane at most marks a segment entry.
template <int MODE>
__device__ __forceinline__ void probe_small(const GraphView& g, const Src& I, uint32_t q,
                                            const uint64_t* keys, uint8_t* mark,
                                            uint32_t* hitpos) {
    static_assert(kSmallLanes == 4 && kSmallSeg == 8, "two destinations per lane of a quad");
    constexpr uint32_t kRounds = kSmallLanes * kSmallDeg / 16;
    const uint32_t deg = I.deg;
    const uint32_t len = I.hi - I.lo;
    const uint32_t* klo = (const uint32_t*)keys;  // low words: destinations
    const uint32_t dmask = (uint32_t)((1ull << g.L) - 1);
    const uint32_t d0 = klo[2ull * (I.lo + min(2 * q, len - 1))] & dmask;
    const uint32_t d1 = klo[2ull * (I.lo + min(2 * q + 1, len - 1))] & dmask;
    // whole 16-byte groups of a block (B >= 4, so a group stays inside it)
    uint32_t blk[kRounds];
#pragma unroll
    for (uint32_t u = 0; u < kRounds; ++u) {
        const uint32_t sl = min(16 * u + 4 * q, deg - 1);
        blk[u] = I.dir;
        if (I.dcls != kNoDir && 16 * u < deg) blk[u] = g.dir[I.dir + (sl >> g.log2B)];
    }
    uint4 x[kRounds];
#pragma unroll
    for (uint32_t u = 0; u < kRounds; ++u) {
        const uint32_t sl = 16 * u + 4 * q;
        if (sl < deg)
            x[u] = *(const uint4*)(g.pool + (((uint64_t)blk[u] << g.log2B) + (sl & (g.B - 1))));
    }
    const uint32_t d[kSmallSeg] = {quad_get<0>(d0), quad_get<0>(d1), quad_get<1>(d0),
                                   quad_get<1>(d1), quad_get<2>(d0), quad_get<2>(d1),
                                   quad_get<3>(d0), quad_get<3>(d1)};
#pragma unroll
    for (uint32_t u = 0; u < kRounds; ++u) {
        const uint32_t sl = 16 * u + 4 * q;
        if (sl >= deg) break;
        const uint32_t left = deg - sl;  // live slots of this group (4 or more: all)
#pragma unroll
        for (uint32_t j = 0; j < kSmallSeg; ++j) {
            if (j >= len) break;
            uint32_t h = 4;
            h = left > 3 && x[u].w == d[j] ? 3u : h;
            h = left > 2 && x[u].z == d[j] ? 2u : h;
            h = left > 1 && x[u].y == d[j] ? 1u : h;
            h = x[u].x == d[j] ? 0u : h;
            if (h == 4) continue;
            if (MODE != kQuery && MODE != kLocate && j > 0 && d[j] == d[j - 1])
                continue;  // not a first occurrence
            mark[I.lo + j] = 1;
            if (MODE == kDelete || MODE == kLocate) hitpos[I.lo + j] = sl + h;
        }
    }
}

// Small items first, then the work items, a wave each.  An item's descriptor
// is the same for the whole wave and lives in scalar registers; a lane takes
// four consecutive slots of a block per step (two when the item has at most
// 128), one directory entry and one load.  A wave's items run in a pipeline:
// while one is searched, the slots and segment samples of the next are in
// flight, the directory entries of the one after it and the descriptor of the
// third, so that the chain descriptor -> directory -> slots costs an item's
// search each, not its latency.  The loads carry no arithmetic on their
// results: a mask there made the wave wait for them where they are issued.
//
// Bound: the searches' instructions and LDS latency, hidden by eight waves per
// SIMD; the slots alone would take 16 us of the 43 and 72 of the 228.  Lane
// groups of 16 to 64 with one item each, without the pipeline, took
// (edge queries, 10^6 of a 2^20-vertex R-MAT graph / 10^7 of a 2^22 one) 71 and
// 430 us, with it 59 and 345; a wave per item at seven waves per SIMD 56 and
// 348, at eight and 128 staged entries 43 and 228 (64 entries 44 and 235,
// 256 entries, which spills, 45 and 259).  Inserts of 10^7: 236 -> 180,
// deletes 453 -> 273.  Comparing every slot with every entry of a short
// segment (4, 8, 16 entries) was no faster than its search.
// VEC: blocks hold whole groups of four slots (B >= 4)
template <int MODE, bool VEC>
__global__ __launch_bounds__(kThreads, kProbeWaves) void k_probe(GraphView g, const uint64_t* keys,
                                                    const BatchCtr* bc, const Item* items,
                                                    const Src* srcs, uint8_t* mark,
                                                    uint32_t* hitpos) {
    constexpr int U = 4;
    constexpr uint32_t kStep = 64 * U;  // slots per wave and step
    constexpr int Q = VEC ? 1 : U;      // directory entries per lane and step
    __shared__ uint32_t stage[kWaves][kStage + 1];  // (a hit reads the entry after its own)
    // the batch's counters, read together
    const unsigned long long alloc = bc->alloc, key_sum = bc->key_sum;
    const uint32_t nohash = bc->nohash;
    const unsigned long long stripe =
        MODE == kInsert || MODE == kDelete ? bc->stripe[lane_id()][kStripeHash] : 0ull;
    if (batch_failed(g.ctr)) return;
    if (MODE == kInsert || MODE == kDelete) {
        // the sorted keys must be the packed keys: their mix64 sums agree
        // (per-workgroup sums of the segments kernel in 64 stripes; one load a lane)
        if (wave_sum(stripe) != key_sum && !nohash) {
            if (lane_id() == 0) g.ctr->err_order = 3;
            return;
        }
    }
    {
        // small items first, kSmallLanes consecutive lanes per touched source
        const uint64_t nq = (uint64_t)(uint32_t)(alloc >> 32) * kSmallLanes;
        const uint64_t stride = (uint64_t)gridDim.x * kThreads;
        for (uint64_t k = (uint64_t)blockIdx.x * kThreads + threadIdx.x; k < nq; k += stride) {
            const Src I = srcs[k / kSmallLanes];
            const uint32_t q = (uint32_t)(k % kSmallLanes);
            // (all four lanes: they exchange the segment's destinations)
            if (small_item(g.B, I.deg, I.hi - I.lo))
                probe_small<MODE>(g, I, q, keys, mark, hitpos);
        }
    }
    const uint32_t nitems = __builtin_amdgcn_readfirstlane((uint32_t)alloc);
    const uint32_t lane = lane_id();
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t nw = gridDim.x * kWaves;
    const uint32_t dmask = (uint32_t)((1ull << g.L) - 1);
    // Where both kinds fit the grid's waves, items go to the last waves, so that
    // no wave has both (10^3 pairs 7.0 -> 6.1 us); beyond that the last waves,
    // which start last, would have two items (10^6 pairs 49 -> 57).
    const uint32_t mine = blockIdx.x * kWaves + wave;
    const uint64_t small = ((alloc >> 32) * kSmallLanes + 63) / 64;
    uint32_t it = __builtin_amdgcn_readfirstlane(nitems + small <= nw ? nw - 1 - mine : mine);
    if (it >= nitems) return;
    uint32_t* st = stage[wave];
    const uint32_t sbase = wave * (uint32_t)sizeof(stage[0]);
    constexpr int kSv = kStage / 64;
    // an item's descriptor, a word per lane, and its fields
    static_assert(sizeof(Item) == 24, "six words");
    auto desc = [&](uint64_t i) {
        return ((const uint32_t*)(items + min(i, (uint64_t)nitems - 1)))[min(lane, 5u)];
    };
    struct Fields {
        uint32_t s0, s1, lo, len, dir;
        bool inl;
    };
    auto fields = [](uint32_t w) {
        const uint32_t lo = __builtin_amdgcn_readlane(w, 2);
        return Fields{(uint32_t)__builtin_amdgcn_readlane(w, 0),
                      (uint32_t)__builtin_amdgcn_readlane(w, 1), lo,
                      (uint32_t)__builtin_amdgcn_readlane(w, 3) - lo,
                      (uint32_t)__builtin_amdgcn_readlane(w, 4),
                      __builtin_amdgcn_readlane(w, 5) != 0};
    };
    // slots per lane of an item's first step, and the lane's first slot there
    auto narrow = [](const Fields& I) { return VEC && I.s1 - I.s0 <= kStep / 2; };
    auto first = [&](const Fields& I) {
        return I.s0 + (VEC ? lane * (narrow(I) ? 2u : 4u) : lane);
    };
    // unconditional loads at clamped positions; slots past the item are masked
    // out by the search
    auto load_dir = [&](const Fields& I, uint32_t s, uint32_t (&e)[Q]) {
#pragma unroll
        for (int k = 0; k < Q; ++k)
            e[k] = I.inl ? I.dir : g.dir[I.dir + (min(s + 64u * k, I.s1 - 1) >> g.log2B)];
    };
    auto load_slots = [&](const Fields& I, uint32_t s, const uint32_t (&e)[Q], uint32_t (&x)[U]) {
        if constexpr (VEC) {
            const uint32_t sl = min(s, I.s1 - 1) & ~3u;
            const uint4 v = *(const uint4*)(g.pool + (((uint64_t)e[0] << g.log2B) +
                                                      (sl & (g.B - 1))));
            x[0] = v.x;
            x[1] = v.y;
            x[2] = v.z;
            x[3] = v.w;
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t sl = min(s + 64u * u, I.s1 - 1);
                x[u] = g.pool[((uint64_t)e[u % Q] << g.log2B) + (sl & (g.B - 1))];
            }
        }
    };
    // a segment of fewer than kStage entries goes to LDS whole, of a longer
    // one every 2^shift-th entry
    auto sampling = [](const Fields& I, uint32_t& shift, uint32_t& ns) {
        const uint32_t q = (I.len + kStage - 2) / (kStage - 1);
        shift = q <= 1 ? 0u : 32u - __builtin_clz(q - 1);
        ns = (I.len + (1u << shift) - 1) >> shift;  // < kStage samples
    };
    // (masked to destinations when they are used: here the wait would end the
    // pipeline)
    auto load_samples = [&](const Fields& I, uint32_t (&sv)[kSv]) {
        uint32_t shift, ns;
        sampling(I, shift, ns);
        const uint32_t* klo = (const uint32_t*)(keys + I.lo);
#pragma unroll
        for (int r = 0; r < kSv; ++r)
            if (r * 64u < ns)
                sv[r] = klo[2ull * ((uint64_t)min(lane + r * 64u, ns - 1) << shift)];
    };
    Fields A = fields(desc(it)), B = fields(desc((uint64_t)it + nw));
    uint32_t wC = desc((uint64_t)it + 2ull * nw);
    uint32_t x[U], sv[kSv], eB[Q];
    {
        uint32_t eA[Q];
        load_dir(A, first(A), eA);
        load_samples(A, sv);
        load_dir(B, first(B), eB);
        load_slots(A, first(A), eA, x);
    }
    while (true) {
        uint32_t shift, ns;
        sampling(A, shift, ns);
        const uint32_t steps = 32u - __builtin_clz(ns);  // 2^steps > ns
        // (a wave's LDS accesses are in order: these writes follow the
        // searches of the item before); the searches read st[0, 2^steps) only
#pragma unroll
        for (int r = 0; r < kSv; ++r)
            if (r * 64u < (1u << steps))
                st[lane + r * 64u] = lane + r * 64u < ns ? sv[r] & dmask : 0xFFFFFFFFu;
        // the next items' loads
        const Fields C = fields(wC);
        uint32_t xB[U], svB[kSv], eC[Q];
        load_slots(B, first(B), eB, xB);
        load_samples(B, svB);
        load_dir(C, first(C), eC);
        wC = desc((uint64_t)it + 3ull * nw);
        wave_fence();
        const uint32_t* klo = (const uint32_t*)(keys + A.lo);
        auto search = [&](const auto& y, uint32_t at, auto apart) {
            constexpr int W = sizeof(y) / 4, kApart = decltype(apart)::value;
            probe_search<MODE, W, kApart>(y, at, A.s1, A.lo, A.len, (const char*)stage, sbase,
                                          steps, shift, klo, dmask, mark, hitpos);
        };
        using Next = std::integral_constant<int, 1>;  // a lane's slots adjoin
        using Apart = std::integral_constant<int, VEC ? 1 : 64>;
        if (narrow(A)) {
            const bool odd = lane & 1;
            const uint32_t y[2] = {odd ? x[2] : x[0], odd ? x[3] : x[1]};
            search(y, first(A), Next());
        } else {
            uint32_t s = first(A);
            for (uint32_t left = A.s1 - A.s0;; left -= kStep) {
                // the loads of step k+1 are issued before step k is searched
                // and copied over after it, so they overlap the search
                const bool more = left > kStep;
                uint32_t x2[U];
                if (more) {
                    uint32_t e2[Q];
                    load_dir(A, s + kStep, e2);
                    load_slots(A, s + kStep, e2, x2);
                }
                search(x, s, Apart());
                if (!more) break;
                s += kStep;
#pragma unroll
                for (int u = 0; u < U; ++u) x[u] = x2[u];
            }
        }
        if ((uint64_t)it + nw >= nitems) break;
        it += nw;
        A = B;
        B = C;
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = xB[u];
#pragma unroll
        for (int r = 0; r < kSv; ++r) sv[r] = svB[r];
#pragma unroll
        for (int k = 0; k < Q; ++k) eB[k] = eC[k];
    }
}

// ------------------------------------------------------------------ plan
__device__ __forceinline__ void plan_insert(const GraphView& g, const BatchCtr* bc, uint64_t n,
                                            uint32_t applied, int sticky);
__device__ __forceinline__ void plan_delete(const GraphView& g, const BatchCtr* bc, uint64_t n,
                                            uint32_t applied);

// a source that one lane compacts by itself
__device__ __forceinline__ bool lane_compactable(uint32_t r, uint32_t lo, uint32_t hi) {
    return r <= kLaneR && hi - lo <= kLaneSeg;
}

// Kept pairs (insert: mark 0) or hits (delete: mark 1) of positions [a, b), by
// one wave.
template <bool INS>
__device__ __forceinline__ uint32_t wave_count(const uint8_t* mark, uint64_t a, uint64_t b) {
    uint32_t c = 0;
    for (uint64_t p = a + lane_id(); p < b; p += 64) c += INS ? mark[p] == 0 : mark[p] != 0;
    return wave_sum(c);
}

// words that other workgroups of the same kernel add to or write
template <typename V>
__device__ __forceinline__ V ld_agent(const V* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The same of a tile inside a segment, by one lane: the tile publishes its
// own count (tkept).  A tile like that waits for nothing and workgroups start
// in order, so it comes; a wait that runs out all the same counts the marks
// here (words of four, each 0 or 1).
constexpr uint32_t kPlanSpins = 1u << 14;
template <bool INS>
__device__ __forceinline__ uint32_t inner_count(const uint32_t* tkept, const uint8_t* mark,
                                                uint64_t tile, uint32_t tl) {
    for (uint32_t spins = 0; spins < kPlanSpins; ++spins) {
        const uint32_t x = ld_agent(tkept + tile);
        if (x) return x - 1u;
        __builtin_amdgcn_s_sleep(4);
    }
    const uint32_t* m = (const uint32_t*)(mark + (tile << tl));
    const uint32_t words = 1u << (tl - 2);
    uint32_t hits = 0;
    for (uint32_t i = 0; i < words; ++i) hits += (uint32_t)__popc(m[i]);
    return INS ? (1u << tl) - hits : hits;
}

// What every touched source of a tile needs: its kept pairs or hits r, then
// (insert) its blocks and directory request, or (delete) its freed blocks and
// who compacts it.  The tile's blocks and listed sources are placed with one
// atomic on the batch's demand; the last tile to finish runs the batch's
// plan.  The words the plan adds up are written by returning atomics only, so
// every tile's share is in them once its `done` is counted, and no fence is
// needed.  A segment that runs past the tile is counted by its head's tile
// (insert: which also leaves the running count to the further tiles): one wave
// per further tile, or, where that would take several rounds, a thread per
// tile that reads the count which the tile itself published; only the last,
// which the segment may end inside of, is still counted here.  (10^6 stored
// pairs of one vertex inserted again, 489 tiles: 449 us for the batch by waves
// alone, now 166.)
//
// Bound: latency (marks, then source records: both streams).  It replaces a
// scan over the pairs, a kernel over the sources and a scan over them
// (insert: 19 -> 6.8 us at 10^4 pairs, 46 -> 18 at 10^6), or a scan over the
// sources that read their records anew and two hit counters kept by the probe
// (delete: 8.3 -> 6.3 us, with the counters and a last kernel of 3.4 us gone).
// All of a thread's sources are read together and placed by one scan (deletes
// of 10^6 pairs 25 -> 16 us, of 10^7 93 -> 60, inserts 26 -> 18 and 76 -> 52;
// a line of its own for each class's requests made inserts 4 and 8 us slower).
template <bool INS, int T, uint32_t R>
__global__ __launch_bounds__(T, 8) void k_plan(GraphView g, uint64_t n, BatchCtr* bc, uint32_t tl,
                                            const uint8_t* mark, Src* srcs, const uint2* tiles,
                                            uint2* carry, uint32_t* tbase, uint32_t* tkept,
                                            uint32_t* t_dreq,
                                            uint32_t* t_drank, uint32_t* list, uint32_t* list2,
                                            int sticky) {
    constexpr uint32_t kTile = T * R;
    __shared__ uint32_t s_pre[kTile + 1];
    __shared__ uint32_t s_cnt[R * T / 64];
    __shared__ unsigned long long s_scan[R * T / 64];
    __shared__ uint32_t lcnt[kMaxClass], lbase[kMaxClass];
    __shared__ uint32_t s_tail[T / 64], s_at2;
    __shared__ unsigned long long s_demand, s_done;
    const uint32_t t = threadIdx.x, w = t >> 6;
    const uint64_t p0 = (uint64_t)blockIdx.x << tl;
    const uint32_t tile = 1u << tl;
    // read before the batch's counters have arrived, at positions inside the
    // buffers
    const uint2 td = tiles[blockIdx.x];
    uint8_t m[R];
#pragma unroll
    for (uint32_t j = 0; j < R; ++j)
        m[j] = mark[min(p0 + min(j * T + t, tile - 1), n - 1)];
    // (an order check that failed leaves nothing to plan)
    const uint64_t lim = batch_failed(g.ctr) ? 0ull : min((uint64_t)bc->n_valid, n);
    const uint32_t np = p0 < lim ? (uint32_t)min((uint64_t)tile, lim - p0) : 0u;
    if (t < kMaxClass) lcnt[t] = 0;
    uint32_t changed = 0;
    if (np) {  // uniform over the workgroup
        const uint32_t t0 = td.x, nh = td.y;
        // the first row's sources and the last one, while the marks are ranked
        const Src row0 = srcs[t0 + (nh ? min(t, nh - 1) : 0u)];
        const uint2 last = *(const uint2*)&srcs[t0 + (nh ? nh - 1 : 0u)];  // lo, hi
        bool f[R];
        uint32_t rank[R];
#pragma unroll
        for (uint32_t j = 0; j < R; ++j)
            f[j] = j * T + t < np && (INS ? m[j] == 0 : m[j] != 0);
        const uint32_t tot = tile_ranks<T>(f, rank, s_cnt);
#pragma unroll
        for (uint32_t j = 0; j < R; ++j) {
            const uint32_t p = j * T + t;
            if (p < np) s_pre[p] = rank[j];
        }
        if (t == 0) {
            s_pre[np] = tot;
            if (!nh)
                __hip_atomic_store(tkept + blockIdx.x, tot + 1u, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
        }
        changed = tot;
        __syncthreads();
        // the rest of a segment that runs past the tile
        uint32_t tail = 0;
        const uint64_t pe = p0 + np;
        if (nh) {
            const uint32_t last_lo = last.x, last_hi = last.y;
            if (last_hi > pe) {
                const uint32_t in_tile = tot - s_pre[last_lo - (uint32_t)p0];
                const uint64_t b1 = ((uint64_t)last_hi - 1) >> tl;
                uint64_t b = blockIdx.x + 1;
                if (b1 - b >= T / 64) {
                    for (; b < b1; b += T) {
                        const uint64_t mb = b + t;
                        uint32_t c[1] = {0}, before[1];
                        if (mb < b1) c[0] = inner_count<INS>(tkept, mark, mb, tl);
                        const uint32_t all = tile_sums<T>(c, before, s_tail);
                        if (INS && mb < b1)
                            carry[mb] = make_uint2(t0 + nh - 1, in_tile + tail + before[0]);
                        tail += all;
                        __syncthreads();
                    }
                    b = b1;
                }
                for (; b <= b1; b += T / 64) {
                    const uint64_t mb = b + w;
                    uint32_t c = 0;
                    if (mb <= b1)
                        c = wave_count<INS>(mark, mb << tl,
                                            min((uint64_t)last_hi, (mb + 1) << tl));
                    if (lane_id() == 0) s_tail[w] = c;
                    __syncthreads();
                    uint32_t before = 0, all = 0;
                    for (uint32_t i = 0; i < T / 64; ++i) {
                        const uint32_t x = s_tail[i];
                        before += i < w ? x : 0u;
                        all += x;
                    }
                    if (INS && mb <= b1 && lane_id() == 0)
                        carry[mb] = make_uint2(t0 + nh - 1, in_tile + tail + before);
                    tail += all;
                    __syncthreads();
                }
            }
        }
        // The sources: blocks (bits 0-31), listed sources (from bit 32) and
        // sources of list2 (from bit 48) of the tile.  All of a thread's
        // sources at once: read, then one scan.
        Src x[R];
        uint32_t cls[R], lrank[R];
        unsigned long long add[R], ex[R];
#pragma unroll
        for (uint32_t j = 0; j < R; ++j)
            x[j] = j == 0 ? row0 : srcs[t0 + (nh ? min(j * T + t, nh - 1) : 0u)];
#pragma unroll
        for (uint32_t j = 0; j < R; ++j) {
            const uint32_t h = j * T + t;
            cls[j] = kNoDir;
            lrank[j] = 0;
            add[j] = 0;
            if (h >= nh) continue;
            const uint32_t r = s_pre[(uint32_t)(min((uint64_t)x[j].hi, pe) - p0)] -
                               s_pre[x[j].lo - (uint32_t)p0] + (h + 1 == nh ? tail : 0u);
            x[j].r = r;
            uint32_t need = 0;
            bool listed = false, second = false;
            if (INS) {
                const uint32_t nb0 = nblocks(g, x[j].deg), nb1 = nblocks(g, x[j].deg + r);
                const uint64_t cap0 = x[j].dcls == kNoDir ? 1ull : (1ull << x[j].dcls);
                if (nb1 > cap0) {
                    cls[j] = ceil_log2(nb1);
                    lrank[j] = atomicAdd(&lcnt[cls[j]], 1u);
                }
                need = nb1 - nb0;
                // the source gives back a directory segment
                listed = cls[j] != kNoDir && x[j].dcls != kNoDir;
                // the commit kernel takes this decision from here: its heavy
                // sources' records change while other waves still run the
                // lane loop, so it must not be made again there
                second = (cls[j] != kNoDir && nb0 > kLaneCopy) || need > kLaneCopy;
                t_dreq[t0 + h] = cls[j] | (second ? kHeavy : 0u);
            } else if (r) {
                need = nblocks(g, x[j].deg) - nblocks(g, x[j].deg - r);
                listed = r <= kBigR && !lane_compactable(r, x[j].lo, x[j].hi);
                second = r > kBigR;
            }
            add[j] = (unsigned long long)need | (unsigned long long)listed << 32 |
                     (unsigned long long)second << 48;
        }
        const unsigned long long run = tile_sums<T>(add, ex, s_scan);
        const uint32_t n2 = (uint32_t)(run >> 48);
        constexpr unsigned long long kLow48 = (1ull << 48) - 1;
        if (t == 0) {
            s_demand = run & kLow48 ? atomicAdd(&bc->demand, run & kLow48) : 0ull;
            tbase[blockIdx.x] = (uint32_t)s_demand;
        }
        if (t == 64) s_at2 = n2 ? atomicAdd(INS ? &bc->n_heavy : &bc->n_big, n2) : 0u;
        if (INS && t >= 128 && t < 128 + kMaxClass) {
            const uint32_t c = lcnt[t - 128];
            lbase[t - 128] = c ? atomicAdd(&g.ctr->dreq[t - 128], c) : 0u;
        }
#pragma unroll
        for (uint32_t j = 0; j < R; ++j)
            if (j * T + t < nh) {
                Src* to = srcs + t0 + j * T + t;
                to->r = x[j].r;
                to->need = (uint32_t)ex[j];
            }
        __syncthreads();
        const uint32_t lb = (uint32_t)(s_demand >> 32), lb2 = s_at2;
#pragma unroll
        for (uint32_t j = 0; j < R; ++j) {
            const uint32_t at = t0 + j * T + t;
            if (add[j] >> 32 & 1) list[lb + ((uint32_t)(ex[j] >> 32) & 0xFFFFu)] = at;
            if (add[j] >> 48) list2[lb2 + (uint32_t)(ex[j] >> 48)] = at;
            if (INS && cls[j] != kNoDir) t_drank[at] = lbase[cls[j]] + lrank[j];
        }
    }
    if (t == 0) s_done = atomicAdd(&bc->done, (1ull << 32) + changed) + (1ull << 32) + changed;
    __syncthreads();
    if (s_done >> 32 == gridDim.x && t < 64) {
        if (INS) plan_insert(g, bc, n, (uint32_t)s_done, sticky);
        else plan_delete(g, bc, n, (uint32_t)s_done);
    }
}

// Allocation plan for the whole batch, one wave (a lane per directory class):
// capacity is checked before any state is written, so a failing batch leaves
// the graph unchanged.  Run by the first wave of the last tile planned.
__device__ __forceinline__ void plan_insert(const GraphView& g, const BatchCtr* bc, uint64_t n,
                                            uint32_t applied, int sticky) {
    DevCounters* c = g.ctr;
    const uint32_t k = lane_id();
    if (batch_failed(c)) {
        // nothing is committed; commit and release see the error
        if (k == 0) c->err_batch = GV_EDEVICE;
        return;
    }
    const bool cl = k < kMaxClass;
    const unsigned long long N = ld_agent(&bc->demand) & 0xffffffffull;
    const unsigned long long free0 = c->free_cnt, bump0 = c->bump;
    const unsigned long long ff = N < free0 ? N : free0;
    const unsigned long long fb = N - ff;
    const uint32_t req = cl ? ld_agent(&c->dreq[k]) : 0u;
    const uint32_t have = cl ? c->dfree_cnt[k] : 0u;
    const uint32_t dff = req < have ? req : have;
    const unsigned long long grow = cl ? (unsigned long long)(req - dff) << k : 0ull;
    const unsigned long long gincl = wave_incl_scan(grow);
    const unsigned long long db0 = c->dir_bump;
    const unsigned long long db_end = db0 + wave_read(gincl, 63);
    const bool ok = bump0 + fb <= g.cap_blocks && db_end <= g.dir_cap;
    if (cl) {
        c->plan_dff[k] = dff;
        c->plan_dbump[k] = db0 + gincl - grow;
        c->dreq[k] = 0;
        if (ok) {
            c->plan_dtop[k] = have;
            c->dfree_cnt[k] = have - dff;
        }
    }
    const unsigned long long live = wave_sum(cl ? (unsigned long long)req << k : 0ull);
    const unsigned long long nuniq = wave_sum(bc->stripe[k][kStripeUniq]);
    const unsigned long long blocks = wave_sum(bc->stripe[k][kStripeBlocks]);
    if (k != 0) return;
    const unsigned long long nv = min((uint64_t)bc->n_valid, n);
    c->c_batches[kInsert] += 1;
    c->c_pairs[kInsert] += n;
    c->c_touched[kInsert] += bc->alloc >> 32;
    c->c_scanned[kInsert] += blocks << g.log2B;
    c->err_batch = 0;
    if (!ok) {
        c->err_batch = GV_ENOMEM;
        if (sticky && !c->err_sticky) c->err_sticky = GV_ENOMEM;
        c->st_applied = c->st_rejected = c->st_dups = 0;
        return;
    }
    c->plan_free_top = free0;
    c->plan_from_free = ff;
    c->plan_bump0 = bump0;
    c->free_cnt = free0 - ff;
    c->bump = bump0 + fb;
    c->dir_bump = db_end;
    c->dir_live += live;
    c->st_applied = applied;
    c->st_rejected = n - nv;
    c->st_dups = nv - nuniq;
    c->c_new_blocks += N;
    c->c_written += applied;
    c->live_edges += applied;
}

// The free-list places and the statistics of a delete batch, one wave.
__device__ __forceinline__ void plan_delete(const GraphView& g, const BatchCtr* bc, uint64_t n,
                                            uint32_t applied) {
    DevCounters* c = g.ctr;
    const uint32_t k = lane_id();
    if (batch_failed(c)) {
        if (k == 0) c->err_batch = GV_EDEVICE;
        return;
    }
    const unsigned long long nuniq = wave_sum(bc->stripe[k][kStripeUniq]);
    const unsigned long long blocks = wave_sum(bc->stripe[k][kStripeBlocks]);
    if (k != 0) return;
    const unsigned long long nv = min((uint64_t)bc->n_valid, n);
    const unsigned long long freed = ld_agent(&bc->demand) & 0xffffffffull;
    c->err_batch = 0;
    c->plan_free_top = c->free_cnt;  // the compaction pushes above it
    c->free_cnt += freed;
    c->st_applied = applied;
    c->st_rejected = n - nv;
    c->st_dups = nv - nuniq;
    c->c_batches[kDelete] += 1;
    c->c_pairs[kDelete] += n;
    c->c_touched[kDelete] += bc->alloc >> 32;
    c->c_scanned[kDelete] += blocks << g.log2B;
    c->c_freed_blocks += freed;
    c->live_edges -= applied;
}

// ------------------------------------------------------------------ insert
// id of the p-th block the batch allocates (free-list top first, then bump)
__device__ __forceinline__ uint32_t planned_block(const GraphView& g, const DevCounters* c,
                                                  uint64_t p) {
    return p < c->plan_from_free ? g.free_stack[c->plan_free_top - 1 - p]
                                 : (uint32_t)(c->plan_bump0 + (p - c->plan_from_free));
}

__device__ __forceinline__ uint32_t planned_segment(const GraphView& g, const DevCounters* c,
                                                    uint32_t cls, uint32_t rk) {
    return rk < c->plan_dff[cls]
               ? g.dfree[g.dfree_base[cls] + c->plan_dtop[cls] - 1 - rk]
               : (uint32_t)(c->plan_dbump[cls] + ((unsigned long long)(rk - c->plan_dff[cls]) << cls));
}

// A source's new blocks and directory: a lane for a source that copies and
// adds at most kLaneCopy entries.
__device__ __forceinline__ void grow_lane(const GraphView& g, const DevCounters* c, const Src& x,
                                          uint64_t p0, uint32_t cls, uint32_t rk,
                                          uint32_t* t_dold, uint32_t* t_doldc, uint32_t t) {
    const VRec r{x.deg, x.dir, x.dcls, 0u};
    const uint32_t nb0 = nblocks(g, x.deg), nb1 = nblocks(g, x.deg + x.r);
    VRec nr = r;
    nr.deg = x.deg + x.r;
    if (cls != kNoDir) {
        const uint32_t off = planned_segment(g, c, cls, rk);
        // (a record keeps its segment when its degree drops, down to zero,
        // so nb0 may be 0 here: then entry 0 of the segment is read)
        uint32_t old[kLaneCopy];
#pragma unroll
        for (uint32_t j = 0; j < kLaneCopy; ++j)
            old[j] = block_of(g, r, min(j, nb0 ? nb0 - 1 : 0u));
#pragma unroll
        for (uint32_t j = 0; j < kLaneCopy; ++j)
            if (j < nb0) g.dir[(uint64_t)off + j] = old[j];
        t_dold[t] = r.dir;
        t_doldc[t] = r.dcls;
        nr.dir = off;
        nr.dcls = cls;
    }
    const uint32_t nnew = nb1 - nb0;
    if (nnew) {
        uint32_t ids[kLaneCopy];
#pragma unroll
        for (uint32_t j = 0; j < kLaneCopy; ++j) ids[j] = planned_block(g, c, p0 + min(j, nnew - 1));
#pragma unroll
        for (uint32_t j = 0; j < kLaneCopy; ++j) {
            if (j >= nnew) continue;
            if (nr.dcls == kNoDir) nr.dir = ids[j];  // the only block, inline
            else g.dir[(uint64_t)nr.dir + nb0 + j] = ids[j];
            g.bown[ids[j]] = make_uint2(x.v, nb0 + j);
        }
    }
    g.vt[x.v] = nr;
}

// Commit of an insert, the tiles of the segments kernel: every kept pair is
// written to slot deg + rank of its source, and every source with kept pairs
// gets its new block ids (and, when its block count outgrows its directory
// segment, a new segment holding a copy of the old entries) and its new
// vertex record.  Sources that copy or add more entries than a lane takes,
// listed (and flagged kHeavy) by the plan, are taken by whole waves.  Both
// read the records as they were before the batch from the sources' own
// copies, and only directory entries that the batch does not write, so they
// need no order between them.  One kernel in place of two, each with its own
// pass over flags, ranks and segment starts, took 9.6 us for 10^4 pairs.  Bound:
// latency, keys -> source -> directory entry or free block -> slot; every step
// is issued for all of a thread's pairs at once (10^4 pairs 6.9 -> 5.4 us, 10^7
// 148 -> 97 against pair after pair and scans through LDS).
template <int T, uint32_t R>
__global__ __launch_bounds__(T) void k_commit(GraphView g, const uint64_t* keys, uint64_t n,
                                              const BatchCtr* bc, uint32_t tl,
                                              const uint8_t* mark, const Src* srcs,
                                              const uint2* tiles, const uint2* carry,
                                              const uint32_t* tbase, const uint32_t* t_dreq,
                                              const uint32_t* t_drank, uint32_t* t_dold,
                                              uint32_t* t_doldc, const uint32_t* heavy) {
    constexpr uint32_t kTile = T * R;
    __shared__ uint32_t s_pre[kTile];
    __shared__ uint32_t s_cnt[R * T / 64], s_cnt2[R * T / 64];
    const DevCounters* c = g.ctr;
    const uint32_t t = threadIdx.x;
    const uint64_t p0 = (uint64_t)blockIdx.x << tl;
    const uint32_t L = g.L;
    const uint32_t tile = 1u << tl;
    // read before the batch's counters have arrived, at positions inside the
    // buffers
    const uint2 td = tiles[blockIdx.x], cr = carry[blockIdx.x];
    uint64_t k[R], q[R];
    uint8_t m[R];
#pragma unroll
    for (uint32_t j = 0; j < R; ++j) {
        const uint64_t i = min(p0 + min(j * T + t, tile - 1), n - 1);
        k[j] = keys[i];
        q[j] = keys[i ? i - 1 : 0];
        m[j] = mark[i];
    }
    if (c->err_batch) return;
    const uint64_t lim = min((uint64_t)bc->n_valid, n);
    if (p0 < lim) {  // uniform over the workgroup
        const uint32_t np = (uint32_t)min((uint64_t)tile, lim - p0);
        const uint32_t t0 = td.x, nh = td.y, base0 = tbase[blockIdx.x];
        // the first of the sources that a thread grows, while the pairs are ranked
        const uint32_t h0 = t0 + (nh ? min(t, nh - 1) : 0u);
        const Src row0 = srcs[h0];
        const uint32_t req0 = t_dreq[h0];
        bool head[R], kept[R];
        uint32_t hr[R], kr[R];
#pragma unroll
        for (uint32_t j = 0; j < R; ++j) {
            const uint32_t p = j * T + t;
            head[j] = p < np && (p0 + p == 0 || (k[j] >> L) != (q[j] >> L));
            kept[j] = p < np && m[j] == 0;
        }
        tile_ranks<T>(head, hr, s_cnt);
        tile_ranks<T>(kept, kr, s_cnt2);
#pragma unroll
        for (uint32_t j = 0; j < R; ++j) s_pre[j * T + t] = kr[j];
        __syncthreads();
        // The rows' sources, then their blocks, then the slots: every step
        // reads for all rows at once, a pair that is not kept something in
        // its place.
        uint32_t lo[R], deg[R], dir[R], dcls[R], need[R], pb[R], h[R];
#pragma unroll
        for (uint32_t j = 0; j < R; ++j) {
            h[j] = hr[j] + (head[j] ? 1u : 0u);  // heads up to this position
            // (none: a segment that began in an earlier tile)
            const Src x = srcs[!kept[j] ? h0 : h[j] ? t0 + h[j] - 1 : cr.x];
            lo[j] = kept[j] ? x.lo : (uint32_t)p0;
            deg[j] = x.deg;
            dir[j] = x.dir;
            dcls[j] = x.dcls;
            need[j] = x.need;
        }
        uint32_t blk[R];
#pragma unroll
        for (uint32_t j = 0; j < R; ++j) pb[j] = tbase[lo[j] >> tl];
#pragma unroll
        for (uint32_t j = 0; j < R; ++j) {
            const uint32_t rank = h[j] ? kr[j] - s_pre[kept[j] ? lo[j] - (uint32_t)p0 : 0u]
                                       : cr.y + kr[j];
            const uint32_t nb0 = nblocks(g, deg[j]);
            deg[j] += rank;  // the slot
            const uint32_t b = deg[j] >> g.log2B;
            // an entry of the directory, the only block, a block of the free
            // list or one past the pool's bump pointer
            const uint64_t p = (uint64_t)pb[j] + need[j] + (b - nb0);
            const bool old = b < nb0, inl = dcls[j] == kNoDir, fl = p < c->plan_from_free;
            const uint32_t* at = (const uint32_t*)keys;
            if (kept[j] && old && !inl) at = g.dir + (uint64_t)dir[j] + b;
            if (kept[j] && !old && fl) at = g.free_stack + (c->plan_free_top - 1 - p);
            const uint32_t v = *at;
            blk[j] = old ? (inl ? dir[j] : v)
                         : (fl ? v : (uint32_t)(c->plan_bump0 + (p - c->plan_from_free)));
        }
#pragma unroll
        for (uint32_t j = 0; j < R; ++j) {
            if (!kept[j]) continue;
            const uint64_t sa = ((uint64_t)blk[j] << g.log2B) + (deg[j] & (g.B - 1));
            g.pool[sa] = (uint32_t)(k[j] & ((1ull << L) - 1));
            attr_zero(g, sa);
        }
        for (uint32_t h = t; h < nh; h += T) {
            const Src x = h == t ? row0 : srcs[t0 + h];
            const uint32_t req = h == t ? req0 : t_dreq[t0 + h];
            if (!x.r || (req & kHeavy)) continue;
            const uint32_t cls = req & kClassMask;
            const uint32_t rk = cls != kNoDir ? t_drank[t0 + h] : 0u;
            grow_lane(g, c, x, (uint64_t)base0 + x.need, cls, rk, t_dold, t_doldc, t0 + h);
        }
    }
    const uint32_t nh = bc->n_heavy, lane = lane_id();
    const uint32_t nw = gridDim.x * (T / 64);
    for (uint32_t i = blockIdx.x * (T / 64) + (t >> 6); i < nh; i += nw) {
        const uint32_t ts = heavy[i];
        const Src x = srcs[ts];
        const VRec r{x.deg, x.dir, x.dcls, 0u};
        const uint32_t nb0 = nblocks(g, r.deg), nb1 = nblocks(g, r.deg + x.r);
        const uint32_t cls = t_dreq[ts] & kClassMask;
        VRec nr = r;
        nr.deg = r.deg + x.r;
        if (cls != kNoDir) {
            const uint32_t off = planned_segment(g, c, cls, t_drank[ts]);
            for (uint32_t j = lane; j < nb0; j += 64) g.dir[(uint64_t)off + j] = block_of(g, r, j);
            if (lane == 0) {
                t_dold[ts] = r.dir;
                t_doldc[ts] = r.dcls;
            }
            nr.dir = off;
            nr.dcls = cls;
        }
        const uint64_t pb = (uint64_t)tbase[x.lo >> tl] + x.need;
        for (uint32_t j = nb0 + lane; j < nb1; j += 64) {
            const uint32_t blk = planned_block(g, c, pb + (j - nb0));
            g.dir[(uint64_t)nr.dir + j] = blk;
            g.bown[blk] = make_uint2(x.v, j);
        }
        if (lane == 0) g.vt[x.v] = nr;
    }
}

// Old directory segments of the sources that moved go on the per-class free
// lists (after the commit kernel has taken its segments from them).
__global__ __launch_bounds__(kThreads) void k_final_ins(GraphView g, const BatchCtr* bc,
                                                        const uint32_t* rel,
                                                        const uint32_t* t_dold,
                                                        const uint32_t* t_doldc) {
    __shared__ uint32_t lcnt[kMaxClass];
    __shared__ uint32_t lbase[kMaxClass];
    __shared__ unsigned long long lfreed;
    const uint32_t nrel = g.ctr->err_batch ? 0u : (uint32_t)(bc->demand >> 32);
    for (uint32_t base = blockIdx.x * kThreads; base < nrel; base += gridDim.x * kThreads) {
        if (threadIdx.x < kMaxClass) lcnt[threadIdx.x] = 0;
        if (threadIdx.x == 0) lfreed = 0;
        __syncthreads();
        const uint32_t k = base + threadIdx.x;
        uint32_t oc = kNoDir, lrank = 0, old = 0;
        if (k < nrel) {
            const uint32_t t = rel[k];
            oc = t_doldc[t];
            old = t_dold[t];
            lrank = atomicAdd(&lcnt[oc], 1u);
            atomicAdd(&lfreed, 1ull << oc);
        }
        __syncthreads();
        if (threadIdx.x < kMaxClass) {
            const uint32_t c = lcnt[threadIdx.x];
            lbase[threadIdx.x] = c ? atomicAdd(&g.ctr->dfree_cnt[threadIdx.x], c) : 0u;
        }
        if (threadIdx.x == 0 && lfreed)
            atomicAdd(&g.ctr->dir_live, (unsigned long long)(-(long long)lfreed));
        __syncthreads();
        if (oc != kNoDir) g.dfree[g.dfree_base[oc] + lbase[oc] + lrank] = old;
        __syncthreads();
    }
}

// ------------------------------------------------------------------ delete

// Compaction of every touched source with at most kBigR hits: holes below the
// new degree (taken in batch order) receive the survivors found above it (in
// slot order), and emptied blocks go on the free list.  The hit positions say
// which slots of the tail are gone, so the probe writes nothing to the pool
// (a tombstone per hit, 4 bytes each into lines of their own, took as long as
// reading the adjacencies: 258 MB written for 8 * 10^6 hits).  A lane takes a
// source with at most kLaneR hits and a short segment: its hit positions in
// whole 16-byte groups, its tail's one or two blocks (from 8 slots per block
// on) read once.  The others are taken by the whole wave in turn.  Bound: the
// chain tail -> holes -> survivors, and lines of the pool read and written for
// a slot or two (10^6 deletes of a 2^20-vertex graph 42 -> 40 us, 10^7 of a
// 2^22-vertex one 420 -> 353).
__device__ __forceinline__ void compact_body(const GraphView& g, const uint32_t* hitpos,
                                             uint32_t* holes, const BatchCtr* bc,
                                             const Src* srcs, const uint32_t* tbase, uint32_t tl,
                                             const uint32_t* mid, uint32_t vb, uint32_t vg) {
    __shared__ uint32_t s_gone[kWaves][kBigR / 32];
    const uint32_t gwave = (vb * kThreads + threadIdx.x) >> 6;
    const DevCounters* c = g.ctr;
    const uint32_t nT = (uint32_t)(bc->alloc >> 32);
    const uint32_t lane = lane_id();
    const uint64_t below = (1ull << lane) - 1;
    const uint32_t stride = vg * kThreads;
    const unsigned long long fbase = c->plan_free_top;
    const uint32_t bm = g.B - 1;
    unsigned long long moved = 0;
    for (uint32_t base = gwave * 64; base < nT; base += stride) {
        const bool live = base + lane < nT;
        const Src D = srcs[live ? base + lane : nT - 1];
        if (!live || !D.r || !lane_compactable(D.r, D.lo, D.hi)) continue;
        const VRec rec{D.deg, D.dir, D.dcls, 0u};
        const uint32_t d = D.deg, dn = d - D.r;
        // the segment's hit positions: kLaneGroups groups of four from the
        // group that holds lo (the buffer ends on a whole group)
        constexpr uint32_t kLaneGroups = kLaneSeg / 4 + 1;
        uint32_t hp[4 * kLaneGroups];
        const uint32_t w0 = D.lo & ~3u;
#pragma unroll
        for (uint32_t u = 0; u < kLaneGroups; ++u) {
            const uint4 v = *(const uint4*)(hitpos + min(w0 + 4 * u, (D.hi - 1) & ~3u));
            hp[4 * u] = v.x;
            hp[4 * u + 1] = v.y;
            hp[4 * u + 2] = v.z;
            hp[4 * u + 3] = v.w;
        }
        // the tail's values
        uint32_t sv[kLaneR], sb0 = 0, sb1 = 0;
        if (g.log2B >= 3) {
            static_assert(kLaneR <= 8, "the tail lies in two blocks of 8 slots");
            sb0 = block_of(g, rec, dn >> g.log2B);
            sb1 = block_of(g, rec, (d - 1) >> g.log2B);
#pragma unroll
            for (uint32_t k = 0; k < kLaneR; ++k) {
                const uint32_t sl = min(dn + k, d - 1);
                const uint32_t b = (sl >> g.log2B) == (dn >> g.log2B) ? sb0 : sb1;
                sv[k] = g.pool[((uint64_t)b << g.log2B) + (sl & bm)];
            }
        } else {
#pragma unroll
            for (uint32_t k = 0; k < kLaneR; ++k)
                sv[k] = g.pool[slot_addr(g, rec, min(dn + k, d - 1))];
        }
        // holes in batch order, survivors in slot order
        uint32_t hm = 0, gone = 0;
#pragma unroll
        for (uint32_t u = 0; u < 4 * kLaneGroups; ++u) {
            const bool hit = w0 + u >= D.lo && w0 + u < D.hi && hp[u] < d;
            hm |= hit && hp[u] < dn ? 1u << u : 0u;
            gone |= hit && hp[u] >= dn ? 1u << (hp[u] - dn) : 0u;
        }
        uint32_t sm = ((1u << D.r) - 1) & ~gone;  // r <= kLaneR
#pragma unroll
        for (uint32_t k = 0; k < kLaneR; ++k) {
            if (!hm || !sm) break;
            const uint32_t u = __builtin_ctz(hm), w = __builtin_ctz(sm);
            hm &= hm - 1;
            sm &= sm - 1;
            uint32_t slot = hp[0], val = sv[0];
#pragma unroll
            for (uint32_t j = 1; j < 4 * kLaneGroups; ++j) slot = u == j ? hp[j] : slot;
#pragma unroll
            for (uint32_t j = 1; j < kLaneR; ++j) val = w == j ? sv[j] : val;
            const uint64_t da = slot_addr(g, rec, slot);
            g.pool[da] = val;
            if (g.A) attr_move(g, da, slot_addr(g, rec, dn + w));
            ++moved;
        }
        const uint32_t nb0 = nblocks(g, d), nb1 = nblocks(g, dn);
        if (nb1 < nb0) {
            const unsigned long long pb = fbase + tbase[D.lo >> tl] + D.need;
            for (uint32_t j = nb1; j < nb0; ++j) g.free_stack[pb + (j - nb1)] = block_of(g, rec, j);
        }
        VRec nr = rec;
        nr.deg = dn;
        if (nb1 == 0 && nr.dcls == kNoDir) nr.dir = 0;
        g.vt[D.v] = nr;
    }
    // sources with more hits or longer segments, listed by the plan: one wave
    // each
    const uint32_t nmid = (uint32_t)(bc->demand >> 32);
    const uint32_t nw = vg * kWaves;
    uint32_t* sg = s_gone[threadIdx.x >> 6];
    for (uint32_t k = gwave; k < nmid; k += nw) {
        const Src H = srcs[mid[k]];
        const VRec rec{H.deg, H.dir, H.dcls, 0u};
        const uint32_t d = H.deg, dn = d - H.r;
        if (lane < kBigR / 32) sg[lane] = 0u;
        wave_fence();
        uint32_t nh = 0;
        // (the next row is in flight: a segment may be long and hold few hits,
        // one pair 10^6 times, inserted and deleted, 5.29 -> 4.22 ms; four rows
        // at once 2.30, but 10^4 deletes 10.6 -> 11.2 us)
        uint32_t next = hitpos[min(H.lo + lane, H.hi - 1)];
        for (uint32_t p0 = H.lo; p0 < H.hi; p0 += 64) {
            const uint32_t hpv = p0 + lane < H.hi ? next : kNoHit;
            if (p0 + 64 < H.hi) next = hitpos[min(p0 + 64 + lane, H.hi - 1)];
            const bool hole = hpv < dn;
            const uint64_t bal = ballot(hole);
            if (hole) holes[H.lo + nh + popc64(bal & below)] = hpv;
            // (r <= kBigR, so the tail's bits fit)
            if (hpv >= dn && hpv < d) atomicOr(&sg[(hpv - dn) >> 5], 1u << ((hpv - dn) & 31));
            nh += popc64(bal);
        }
        __threadfence_block();
        wave_fence();
        uint32_t ns = 0;
        for (uint32_t s0 = dn; s0 < d; s0 += 64) {
            const uint32_t sl = s0 + lane, o = sl - dn;
            const bool surv = sl < d && !((sg[(sl < d ? o : 0u) >> 5] >> (o & 31)) & 1u);
            uint32_t x = 0;
            if (surv) x = g.pool[slot_addr(g, rec, sl)];
            const uint64_t bal = ballot(surv);
            if (surv) {
                // survivors above dn and holes below it are equal in number;
                // the guards only keep a broken invariant from writing wild
                const uint32_t qq = ns + popc64(bal & below);
                if (qq < nh) {
                    const uint32_t dest = holes[H.lo + qq];
                    if (dest < dn) {
                        const uint64_t da = slot_addr(g, rec, dest);
                        g.pool[da] = x;
                        if (g.A) attr_move(g, da, slot_addr(g, rec, sl));
                    }
                }
            }
            ns += popc64(bal);
        }
        moved += lane == 0 ? ns : 0;
        const uint32_t nb0 = nblocks(g, d), nb1 = nblocks(g, dn);
        const unsigned long long pb = fbase + tbase[H.lo >> tl] + H.need;
        for (uint32_t j = nb1 + lane; j < nb0; j += 64)
            g.free_stack[pb + (j - nb1)] = block_of(g, rec, j);
        if (lane == 0) {
            VRec nr = rec;
            nr.deg = dn;
            if (nb1 == 0 && nr.dcls == kNoDir) nr.dir = 0;
            g.vt[H.v] = nr;
        }
        wave_fence();
    }
    moved = wave_sum(moved);
    if (lane == 0 && moved) atomicAdd(&g.ctr->stripe[gwave & 63][0], moved);
}

// One workgroup per source with more than kBigR hits (hubs), same pairing; the
// slots of the tail that are gone get a tombstone first.
__device__ __forceinline__ void compact_big_body(const GraphView& g, const uint32_t* hitpos,
                                                 uint32_t* holes, const BatchCtr* bc,
                                                 const Src* srcs,
                                                 const uint32_t* tbase, uint32_t tl,
                                                 const uint32_t* big, uint32_t vb,
                                                 uint32_t vg) {
    __shared__ uint32_t lds[kWaves];
    const uint32_t nbig = bc->n_big;
    const unsigned long long fbase = g.ctr->plan_free_top;
    const uint32_t tid = threadIdx.x;
    unsigned long long moved = 0;
    for (uint32_t q = vb; q < nbig; q += vg) {
        const Src D = srcs[big[q]];
        const VRec rec{D.deg, D.dir, D.dcls, 0u};
        const uint32_t d = D.deg, dn = d - D.r;
        uint32_t nh = 0;
        for (uint32_t p0 = D.lo; p0 < D.hi; p0 += kThreads) {
            const uint32_t p = p0 + tid;
            const uint32_t hp = p < D.hi ? hitpos[p] : kNoHit;
            const uint32_t hole = hp < dn;
            if (!hole && hp < d) g.pool[slot_addr(g, rec, hp)] = kTomb;
            uint32_t tot;
            const uint32_t ex = block_excl_scan(hole, lds, tot);
            if (hole) holes[D.lo + nh + ex] = hp;
            nh += tot;
        }
        __threadfence_block();
        __syncthreads();
        uint32_t ns = 0;
        for (uint32_t s0 = dn; s0 < d; s0 += kThreads) {
            const uint32_t s = s0 + tid;
            uint32_t x = kTomb;
            if (s < d) x = g.pool[slot_addr(g, rec, s)];
            const uint32_t surv = x != kTomb;
            uint32_t tot;
            const uint32_t ex = block_excl_scan(surv, lds, tot);
            if (surv) {
                const uint32_t qq = ns + ex;
                if (qq < nh) {
                    const uint32_t dest = holes[D.lo + qq];
                    if (dest < dn) {
                        const uint64_t da = slot_addr(g, rec, dest);
                        g.pool[da] = x;
                        if (g.A) attr_move(g, da, slot_addr(g, rec, s));
                    }
                }
            }
            ns += tot;
        }
        moved += tid == 0 ? ns : 0;
        const uint32_t nb0 = nblocks(g, d), nb1 = nblocks(g, dn);
        const unsigned long long pb = fbase + tbase[D.lo >> tl] + D.need;
        for (uint32_t j = nb1 + tid; j < nb0; j += kThreads)
            g.free_stack[pb + (j - nb1)] = block_of(g, rec, j);
        if (tid == 0) {
            VRec nr = rec;
            nr.deg = dn;
            if (nb1 == 0 && nr.dcls == kNoDir) nr.dir = 0;
            g.vt[D.v] = nr;
        }
        __syncthreads();
    }
    if (tid == 0 && moved) atomicAdd(&g.ctr->stripe[vb & 63][0], moved);
}

// Both compactions in one launch: the first nbig workgroups take the hubs
// (they run longest, so they start first), the rest the other sources.
__global__ __launch_bounds__(kThreads) void k_compact(GraphView g, const uint32_t* hitpos,
                                                      uint32_t* holes,
                                                      const BatchCtr* bc, const Src* srcs,
                                                      const uint32_t* tbase, uint32_t tl,
                                                      const uint32_t* mid, const uint32_t* big,
                                                      uint32_t nbig) {
    if (batch_failed(g.ctr)) return;
    if (blockIdx.x < nbig)
        compact_big_body(g, hitpos, holes, bc, srcs, tbase, tl, big, blockIdx.x, nbig);
    else
        compact_body(g, hitpos, holes, bc, srcs, tbase, tl, mid, blockIdx.x - nbig,
                     gridDim.x - nbig);
}

// ------------------------------------------------------------------ query
__global__ __launch_bounds__(kThreads) void k_answer(GraphView g, const BatchCtr* bc,
                                                     const uint32_t* vals, const uint8_t* mark,
                                                     uint64_t n, uint8_t* out) {
    const uint64_t i = thread_index();
    if (batch_failed(g.ctr)) return;  // the answers are not written; the call reports the error
    const unsigned long long nv = min((uint64_t)bc->n_valid, n);
    if (i < 64) {
        const unsigned long long blocks = wave_sum(bc->stripe[i][kStripeBlocks]);
        if (i == 0) {
            DevCounters* c = g.ctr;
            c->c_batches[kQuery] += 1;
            c->c_pairs[kQuery] += n;
            c->c_touched[kQuery] += bc->alloc >> 32;
            c->c_scanned[kQuery] += blocks << g.log2B;
        }
    }
    if (i < nv && vals[i] < n) out[vals[i]] = mark[i];
}

// ------------------------------------------------------------------ attributes
// get: a found pair's attributes (read at the slot the probe recorded) at
// its input position; a pair not found reads zeros
__global__ __launch_bounds__(kThreads) void k_attr_get(GraphView g, const BatchCtr* bc,
                                                       const uint64_t* keys,
                                                       const uint32_t* vals, const uint8_t* mark,
                                                       const uint32_t* hitpos, uint64_t n,
                                                       uint32_t* out) {
    const uint64_t i = thread_index();
    if (batch_failed(g.ctr)) return;
    const uint64_t nv = min((uint64_t)bc->n_valid, n);
    if (i >= nv || vals[i] >= n) return;
    const uint64_t o = (uint64_t)vals[i] * g.A;
    if (!mark[i]) {
        for (uint32_t k = 0; k < g.A; ++k) out[o + k] = 0u;
        return;
    }
    const uint64_t a = slot_addr(g, g.vt[keys[i] >> g.L], hitpos[i]);
    for (uint32_t k = 0; k < g.A; ++k) out[o + k] = g.apool[a * g.A + k];
}

// set: the last occurrence of each found pair in input order (the sort is
// stable, so the last of its run) writes its attributes; counts for the
// statistics
__global__ __launch_bounds__(kThreads) void k_attr_set(GraphView g, const BatchCtr* bc,
                                                       const uint64_t* keys,
                                                       const uint32_t* vals, const uint8_t* mark,
                                                       const uint32_t* hitpos, uint64_t n,
                                                       const uint32_t* in) {
    __shared__ unsigned long long lds[kWaves];
    const uint64_t i = thread_index();
    if (batch_failed(g.ctr)) return;
    const uint64_t nv = min((uint64_t)bc->n_valid, n);
    if (i == 0) g.ctr->st_valid = nv;
    unsigned long long distinct = 0, applied = 0;
    if (i < nv) {
        const bool last = i + 1 >= nv || keys[i + 1] != keys[i];
        distinct = last;
        if (last && mark[i] && vals[i] < n) {
            applied = 1;
            const uint64_t a = slot_addr(g, g.vt[keys[i] >> g.L], hitpos[i]);
            const uint64_t o = (uint64_t)vals[i] * g.A;
            for (uint32_t k = 0; k < g.A; ++k) g.apool[a * g.A + k] = in[o + k];
        }
    }
    distinct = block_sum(distinct, lds);
    applied = block_sum(applied, lds);
    if (threadIdx.x == 0) {
        if (distinct) atomicAdd(&g.ctr->n_uniq, distinct);
        if (applied) atomicAdd(&g.ctr->st_applied, applied);
    }
}

__global__ void k_attr_begin(DevCounters* c) {
    c->n_uniq = 0;
    c->st_applied = 0;
}

__global__ __launch_bounds__(kThreads) void k_zero_attr(uint32_t* p, uint64_t n) {
    const uint64_t i = thread_index();
    if (i < n) p[i] = 0u;
}

__global__ void k_set_u32(uint32_t* p, uint32_t v) { *p = v; }
__global__ void k_set_u64(unsigned long long* p, unsigned long long v) { *p = v; }

void set_u32(gv_graph* g, uint32_t* p, uint32_t value) {
    g->ctx.launch("set", k_set_u32, 1, 1, p, value);
}

void set_u64(gv_graph* g, unsigned long long* p, unsigned long long value) {
    g->ctx.launch("set", k_set_u64, 1, 1, p, value);
}

// ------------------------------------------------------------------ driver
// Runs f on the probe variant of MODE for blocks of B slots.
template <int MODE, typename F>
static void with_probe(uint32_t B, F&& f) {
    if (B >= 4) return f(k_probe<MODE, true>);
    return f(k_probe<MODE, false>);
}

bool probe_shape_ok(uint32_t group, uint32_t unroll) {
    return (group == 16 || group == 32 || group == 64) && (unroll == 2 || unroll == 4 || unroll == 8);
}

// occupancy lookups of the looping kernels, made before a recording
void edge_batch_warm() {
    auto warm = [](auto kernel) { resident_grid(kernel, kThreads); };
    for (uint32_t B : {1u, 4u}) {
        with_probe<kInsert>(B, warm);
        with_probe<kDelete>(B, warm);
        with_probe<kQuery>(B, warm);
        with_probe<kLocate>(B, warm);
    }
    resident_grid(k_compact, kThreads);
    resident_grid(k_os_pass<uint64_t, false, kPsRounds>, kPsThreads);
    resident_grid(k_os_pass<uint64_t, true, kPsRounds>, kPsThreads);
    resident_grid(k_os_pass<uint64_t, false, kPsRoundsLong>, kPsThreads);
    resident_grid(k_os_pass<uint64_t, false, kPsRoundsShort>, kPsThreads);
    resident_grid(k_os_pass<uint64_t, true, kPsRoundsShort>, kPsThreads);
}

// bytes of g->scratch edge_batch carves for n pairs (edge_batch_sorted carves
// the same)
size_t edge_batch_bytes(const gv_graph* g, EdgeMode mode, uint64_t n) {
    if (n == 0) return 0;
    BatchArrays A;
    Carver m(nullptr);
    carve_batch(m, A, n, n + div_up(g->item_slots, (uint64_t)g->tune.item_chunk) + 1, mode,
                2 * (int)g->v.L);
    return m.used;
}

// Insert and delete batches whose keys arrive sorted (keys[0, *count), the
// count on the device; they come from the library's own sort of a mixed
// list): clears the batch counters, sets the valid count and turns the
// probe's multiset check off (there is no packing to compare with; the
// segments kernel still checks the order).
__global__ __launch_bounds__(kOsThreads) void k_sorted_prep(BatchCtr* bc,
                                                            const unsigned long long* count) {
    const unsigned long long n = *count;
    clear_batch(bc, threadIdx.x, kOsThreads);
    __syncthreads();
    if (threadIdx.x == 0) {
        bc->n_valid = n;
        bc->nohash = 1;
    }
}

// Insert and delete batches of at most this many pairs are sorted by rank: up
// to the tuning's small_sort_max, whose largest value stands for kRankMax,
// where the two ways cross (a batch of 16384 pairs 53 us, of 16385 75).  With the
// sort overlap on, the setting is taken as it stands and larger batches go to
// the side stream.  Called one at a time that pays from about 3 * 10^4 pairs on
// (79 us against 85; 2.6 * 10^5 98 against 126); from 4097 to 16384 pairs it is
// the longer way, 72 to 77 us against 40 to 53.
static uint64_t rank_limit(const gv_graph* g) {
    const uint64_t m = g->tune.small_sort_max;
    return m < kOsTile || g->tune.overlap ? m : kRankMax;
}

static void edge_run(gv_graph* g, EdgeMode mode, const uint32_t* src, const uint32_t* dst,
                     const uint64_t* sorted, const unsigned long long* sorted_n, uint64_t n,
                     uint8_t* out, bool sticky, void* fixed, size_t fixed_bytes,
                     uint8_t* mark_out, const AttrOp* aop = nullptr);

void edge_batch(gv_graph* g, EdgeMode mode, const uint32_t* src, const uint32_t* dst, uint64_t n,
                uint8_t* out, bool sticky, void* fixed, size_t fixed_bytes) {
    edge_run(g, mode, src, dst, nullptr, nullptr, n, out, sticky, fixed, fixed_bytes, nullptr);
}

void edge_batch_sorted(gv_graph* g, EdgeMode mode, const uint64_t* keys,
                       const unsigned long long* count, uint64_t n_max, bool sticky,
                       uint8_t* mark_out) {
    if (mode == kQuery) fail(GV_EINVAL, "sorted batches are inserts or deletes");
    edge_run(g, mode, nullptr, nullptr, keys, count, n_max, nullptr, sticky, nullptr, 0,
             mark_out);
}

void edge_attrs(gv_graph* g, const uint32_t* src, const uint32_t* dst, uint64_t n,
                uint8_t* found, uint32_t* out, const uint32_t* in) {
    if (n == 0) return;
    const AttrOp op{out, in};
    Ctx& c = g->ctx;
    if (out) {
        // answers of invalid pairs are written by the packing scan; their
        // attributes read zeros
        c.launch("attr_get", k_zero_attr, div_up(n * g->v.A, kThreads), kThreads, out,
                 n * g->v.A);
    } else {
        c.launch("attr_set", k_attr_begin, 1, 1, g->v.ctr);
    }
    edge_run(g, kQuery, src, dst, nullptr, nullptr, n, found, true, nullptr, 0, nullptr, &op);
}

void overlap_open(gv_graph* g) {
    gv_graph::Overlap& o = g->ov;
    if (o.stream) return;
    hip_check(hipStreamCreateWithFlags(&o.stream, hipStreamNonBlocking), "hipStreamCreate");
    o.ctx.stream = o.stream;
    hipEvent_t* evs[] = {&o.sorted[0], &o.sorted[1], &o.done[0],    &o.done[1], &o.fence,
                         &o.msorted[0], &o.msorted[1], &o.mdone[0], &o.mdone[1]};
    for (hipEvent_t* e : evs)
        hip_check(hipEventCreateWithFlags(e, hipEventDisableTiming), "hipEventCreate");
}

// the id of the capture the stream is in, 0 when it is not being captured
static unsigned long long capture_id(hipStream_t s) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    unsigned long long id = 0;
    hip_check(hipStreamGetCaptureInfo(s, &st, &id), "hipStreamGetCaptureInfo");
    return st == hipStreamCaptureStatusActive ? id : 0ull;
}

void overlap_capture(gv_graph* g) {
    gv_graph::Overlap& o = g->ov;
    const unsigned long long cap = capture_id(g->ctx.stream);
    if (cap == o.capture) return;
    o.capture = cap;
    o.used[0] = o.used[1] = false;
    o.mused[0] = o.mused[1] = false;
    o.seq = ~0ull;
    o.joined = false;
}

void overlap_fence(gv_graph* g) {
    gv_graph::Overlap& o = g->ov;
    hip_check(hipEventRecord(o.fence, g->ctx.stream), "hipEventRecord");
    hip_check(hipStreamWaitEvent(o.stream, o.fence, 0), "hipStreamWaitEvent");
    o.joined = true;
}

static void edge_run(gv_graph* g, EdgeMode mode, const uint32_t* src, const uint32_t* dst,
                     const uint64_t* sorted, const unsigned long long* sorted_n, uint64_t n,
                     uint8_t* out, bool sticky, void* fixed, size_t fixed_bytes,
                     uint8_t* mark_out, const AttrOp* aop) {
    if (n == 0) return;
    if (n >= 0x3fffffffull) fail(GV_EINVAL, "batch too large");
    if (mode == kInsert) g->edge_bound_host += n;
    Ctx& c = g->ctx;
    const GraphView& v = g->v;
    const uint64_t icap = n + div_up(g->item_slots, (uint64_t)g->tune.item_chunk) + 1;
    const int bits = 2 * (int)v.L;
    // sort overlap: this batch's pack and sort go to the side stream (also
    // while the graph's stream is captured: the side stream then joins the
    // capture through the first wait, and the recording keeps both branches)
    const uint64_t rank_max = mode == kQuery ? kRankMax : rank_limit(g);
    const bool ovb = g->tune.overlap && !sorted && !fixed && mode != kQuery && bits > 0 &&
                     n > rank_max;
    if (ovb) overlap_capture(g);
    const int ob = (int)(g->ov.count & 1);  // its buffer
    BatchArrays A;
    {
        Carver m(nullptr);
        carve_batch(m, A, n, icap, mode, bits);
        void* base = fixed;
        if (fixed) {
            if (m.used > fixed_bytes) fail(GV_ERANGE, "batch does not fit the fixed scratch");
        } else {
            // a buffer that grows first synchronises the graph's stream, and
            // with it every sort queued on the side stream
            Scratch& buf = ovb && ob ? g->ov.scr : g->scratch;
            buf.ensure(m.used, c.stream);
            base = buf.ptr;
        }
        Carver cv(base);
        carve_batch(cv, A, n, icap, mode, bits);
        // a sorted batch's probe writes its per-key result where the caller
        // wants it (n_max bytes)
        if (mark_out && sorted) A.mark = mark_out;
    }
    BatchCtr* bc = A.bc;
    uint32_t* err = &bc->sort_err;
    const unsigned long long* n_valid = &bc->n_valid;
    const uint64_t grid = div_up(n, kThreads);

    bool flip;
    const uint64_t* keys_in = nullptr;
    if (sorted) {
        c.launch("pack", k_sorted_prep, 1, kOsThreads, bc, sorted_n);
        keys_in = sorted;
        flip = false;
    } else if (n <= rank_max) {
        rank_sort(c, "pack", EdgeKeys{v, src, dst, out, bc}, n, A.keys1, A.keys0, A.vals0);
        flip = false;
    } else if (mode == kQuery) {
        // (keys of no bits take no sort, whose first kernel clears the counters
        // that follow n_valid, the scan's total)
        static_assert(offsetof(BatchCtr, n_valid) == 0, "the first word");
        if (bits == 0) c.launch("begin", k_begin, 1, kThreads, bc);
        scan2(c, "pack", PackIn{v, src, dst}, PackOut{v.L, A.keys0, A.vals0, out}, n, A.part,
              &bc->n_valid);
        flip = onesweep<uint64_t, true>(c, A.keys0, A.keys1, A.vals0, A.vals1,
                                        (const uint32_t*)n_valid, n, bits, A.state, err,
                                        g->spin_limit, false, (uint32_t*)bc + 2,
                                        sizeof(BatchCtr) / 4 - 2);
    } else {
        // With the sort overlap the packing and the passes run on the side
        // stream, which reads the pairs and the activity bitmap (which no
        // edge batch changes) and writes only this batch's buffer: it waits
        // for the graph's stream when anything else was queued there since
        // the last overlapped batch, and for the batch that used the buffer
        // before.
        gv_graph::Overlap& o = g->ov;
        if (ovb) {
            overlap_open(g);
            o.ctx.prof = c.prof;
            o.ctx.only = c.only;
            if (c.seq != o.seq) {
                overlap_fence(g);
            } else if (o.used[ob]) {
                // (with a fence, the wait for the graph's stream covers this one)
                hip_check(hipStreamWaitEvent(o.stream, o.done[ob], 0), "hipStreamWaitEvent");
            }
        }
        Ctx& sc = ovb ? o.ctx : c;
        const uint64_t sentinel = bits >= 64 ? ~0ull : (1ull << bits) - 1;
        sc.launch("pack", k_pack_hist, os_hist_groups(n), kOsThreads, v, src, dst, n,
                  bits > 0 ? os_passes(bits) : 0, sentinel, A.keys0, bc, A.state, A.state_words,
                  os_hpart(A.state, n, bits), A.vpart, A.hpart);
        os_hist_sum(sc, A.state, n, bits, (const uint32_t*)A.vpart, &bc->n_valid,
                    (const unsigned long long*)A.hpart, &bc->key_sum);
        flip = onesweep_passes<uint64_t, false>(sc, A.keys0, A.keys1, nullptr, nullptr, nullptr, n,
                                                bits, A.state, err, g->spin_limit, ovb);
        if (ovb) {
            sc.close_run();
            hip_check(hipEventRecord(o.sorted[ob], o.stream), "hipEventRecord");
            hip_check(hipStreamWaitEvent(c.stream, o.sorted[ob], 0), "hipStreamWaitEvent");
        }
    }
    const uint64_t* keys = keys_in ? keys_in : flip ? A.keys1 : A.keys0;
    const uint32_t* vals = flip ? A.vals1 : A.vals0;

    const uint32_t tl = tile_log(n);
    const uint64_t ntiles = div_up(n, 1ull << tl);
    // workgroups of 256 threads while a tile is at most four positions each,
    // and no code for rows that a small tile does not have (a small
    // batch's workgroups each fetch the kernel's instructions anew: segments
    // and plan of 10^3 pairs 1 us less each)
    auto with_threads = [&](auto&& f) {
        using std::integral_constant;
        using One = integral_constant<uint32_t, 1>;
        using Rows = integral_constant<uint32_t, kTileRows>;
        if ((1u << tl) <= kThreads) f(integral_constant<int, kThreads>{}, One{});
        else if ((1u << tl) <= kThreads * kTileRows) f(integral_constant<int, kThreads>{}, Rows{});
        else f(integral_constant<int, 1024>{}, Rows{});
    };
    const uint32_t chunk = g->tune.item_chunk;
    with_threads([&](auto threads, auto rows) {
        constexpr int T = decltype(threads)::value;
        constexpr uint32_t R = decltype(rows)::value;
        c.launch("segments", k_segments<T, R>, ntiles, T, v, keys, n, bc, tl, A.mark,
                 mode == kInsert ? 1 : 0, mode == kDelete ? A.hitpos : nullptr, A.srcs, A.tiles,
                 A.tkept, A.items, icap, chunk);
    });
    const uint64_t pwant = div_up(icap, (uint64_t)kWaves);
    auto probe = [&](auto mode_tag, const char* name, uint32_t* hitpos) {
        constexpr int M = decltype(mode_tag)::value;
        with_probe<M>(v.B, [&](auto kernel) {
            c.launch(name, kernel, std::min<uint64_t>(pwant, resident_grid(kernel, kThreads)),
                     kThreads, v, keys, (const BatchCtr*)bc, (const Item*)A.items,
                     (const Src*)A.srcs, A.mark, hitpos);
        });
    };

    if (mode == kInsert) {
        probe(std::integral_constant<int, kInsert>{}, "probe_insert", nullptr);
        with_threads([&](auto threads, auto rows) {
            constexpr int T = decltype(threads)::value;
            constexpr uint32_t R = decltype(rows)::value;
            c.launch("plan_insert", k_plan<true, T, R>, ntiles, T, v, n, bc, tl,
                     (const uint8_t*)A.mark, A.srcs, (const uint2*)A.tiles, A.carry, A.tbase,
                     A.tkept, A.t_dreq, A.t_drank, A.rel, A.heavy, (int)sticky);
            c.launch("commit", k_commit<T, R>, ntiles, T, v, keys, n, (const BatchCtr*)bc, tl,
                     (const uint8_t*)A.mark, (const Src*)A.srcs, (const uint2*)A.tiles,
                     (const uint2*)A.carry, (const uint32_t*)A.tbase, (const uint32_t*)A.t_dreq,
                     (const uint32_t*)A.t_drank, A.t_dold, A.t_doldc, (const uint32_t*)A.heavy);
        });
        c.launch("final_insert", k_final_ins, std::min<uint64_t>(grid, 64), kThreads, v,
                 (const BatchCtr*)bc, (const uint32_t*)A.rel, (const uint32_t*)A.t_dold,
                 (const uint32_t*)A.t_doldc);
    } else if (mode == kDelete) {
        probe(std::integral_constant<int, kDelete>{}, "probe_delete", A.hitpos);
        with_threads([&](auto threads, auto rows) {
            constexpr int T = decltype(threads)::value;
            constexpr uint32_t R = decltype(rows)::value;
            c.launch("plan_delete", k_plan<false, T, R>, ntiles, T, v, n, bc, tl,
                     (const uint8_t*)A.mark, A.srcs, (const uint2*)A.tiles, (uint2*)nullptr,
                     A.tbase, A.tkept, (uint32_t*)nullptr, (uint32_t*)nullptr, A.heavy, A.big, 0);
        });
        const uint32_t nbig = kBigGroups;
        c.launch("compact", k_compact,
                 nbig + std::min<uint64_t>(div_up(n, kThreads), resident_grid(k_compact, kThreads)),
                 kThreads, v, (const uint32_t*)A.hitpos, A.holes, (const BatchCtr*)bc,
                 (const Src*)A.srcs, (const uint32_t*)A.tbase, tl,
                 (const uint32_t*)A.heavy, (const uint32_t*)A.big, nbig);
    } else if (aop) {
        probe(std::integral_constant<int, kLocate>{}, "probe_locate", A.hitpos);
        if (aop->out) {
            c.launch("answer", k_answer, grid, kThreads, v, (const BatchCtr*)bc, vals,
                     (const uint8_t*)A.mark, n, out);
            c.launch("attr_get", k_attr_get, grid, kThreads, v, (const BatchCtr*)bc, keys, vals,
                     (const uint8_t*)A.mark, (const uint32_t*)A.hitpos, n, aop->out);
        } else {
            c.launch("attr_set", k_attr_set, grid, kThreads, v, (const BatchCtr*)bc, keys, vals,
                     (const uint8_t*)A.mark, (const uint32_t*)A.hitpos, n, aop->in);
        }
    } else {
        probe(std::integral_constant<int, kQuery>{}, "probe_query", nullptr);
        c.launch("answer", k_answer, grid, kThreads, v, (const BatchCtr*)bc, vals,
                 (const uint8_t*)A.mark, n, out);
    }
    if (ovb) {
        gv_graph::Overlap& o = g->ov;
        hip_check(hipEventRecord(o.done[ob], c.stream), "hipEventRecord");
        o.used[ob] = true;
        ++o.count;
        o.seq = c.seq;
    }
}

}  // namespace gv
