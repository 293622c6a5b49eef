// gv_prim.h -- device-wide exclusive scan and stable LSD radix sort for
// wave64 (gfx950), written for this library.
//
// Scan: reduce-then-scan over tiles of kScanTile elements; inputs and outputs
// are functors so that producers and consumers fuse into the scan kernels.
//
// Sort: 8-bit digits, one kernel per pass (below).  Ranking is
// contention-free: the 64 lanes of a wave find the lanes holding the same
// digit with eight ballots (one per digit bit).  Keys keep their input order
// within a digit, so the sort is stable.
#pragma once

#include <algorithm>
#include <type_traits>
#include <utility>

#include "gv_device.h"
#include "gv_host.h"

namespace gv {

constexpr int kScanItems = 8;
constexpr uint64_t kScanTile = (uint64_t)kThreads * kScanItems;
constexpr int kRadixBits = 8;
constexpr int kRadix = 1 << kRadixBits;

template <typename T>
struct ArrOut {
    T* a;
    __device__ void operator()(uint64_t i, T v) const { a[i] = v; }
};

// ------------------------------------------------------------------ scan
template <typename T, typename In>
__global__ __launch_bounds__(kThreads) void k_scan_reduce(In in, uint64_t n, T* partial) {
    __shared__ T lds[kWaves];
    const uint64_t base = (uint64_t)blockIdx.x * kScanTile;
    T s = 0;
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
        uint64_t i = base + (uint64_t)j * kThreads + threadIdx.x;
        if (i < n) s += in(i);
    }
    T tot = block_sum(s, lds);
    if (threadIdx.x == 0) partial[blockIdx.x] = tot;
}

// one workgroup: exclusive scan of the tile sums in place; total -> *total
template <typename T>
__global__ __launch_bounds__(kThreads) void k_scan_partials(T* partial, uint64_t nt, T* total) {
    __shared__ T lds[kWaves];
    T carry = 0;
    for (uint64_t b = 0; b < nt; b += kThreads) {
        uint64_t i = b + threadIdx.x;
        T x = i < nt ? partial[i] : T(0);
        T tot;
        T ex = block_excl_scan(x, lds, tot);
        if (i < nt) partial[i] = carry + ex;
        carry += tot;
    }
    if (threadIdx.x == 0 && total) *total = carry;
}

template <typename T, typename In, typename Out>
__global__ __launch_bounds__(kThreads) void k_scan_down(In in, Out out, uint64_t n, const T* partial) {
    __shared__ T lds[kWaves];
    const uint64_t base = (uint64_t)blockIdx.x * kScanTile;
    T carry = partial[blockIdx.x];
#pragma unroll 1
    for (int j = 0; j < kScanItems; ++j) {
        uint64_t i = base + (uint64_t)j * kThreads + threadIdx.x;
        T x = i < n ? in(i) : T(0);
        T tot;
        T ex = block_excl_scan(x, lds, tot);
        if (i < n) out(i, carry + ex);
        carry += tot;
    }
}

inline uint64_t scan_partials_needed(uint64_t n) { return div_up(n, kScanTile) + 1; }

template <typename T>
__global__ void k_zero_total(T* p) {
    *p = T(0);
}

// Exclusive scan of in(0..n-1) into out(i, prefix); the sum goes to the device
// location `total` when non-null.  `partial` needs scan_partials_needed(n).
template <typename T, typename In, typename Out>
void scan_excl(Ctx& c, In in, Out out, uint64_t n, T* partial, T* total) {
    if (n == 0) {
        // a kernel, not a memset, so that the call can be recorded in a graph
        if (total) c.launch("scan_zero", k_zero_total<T>, 1, 1, total);
        return;
    }
    uint64_t nt = div_up(n, kScanTile);
    c.launch("scan_reduce", k_scan_reduce<T, In>, nt, kThreads, in, n, partial);
    c.launch("scan_partials", k_scan_partials<T>, 1, kThreads, partial, nt, total);
    c.launch("scan_down", k_scan_down<T, In, Out>, nt, kThreads, in, out, n, (const T*)partial);
}

// ------------------------------------------------------------------ sort
// Lanes of this wave that are active and hold the same digit as this lane.
// Four vector instructions per bit: the lane's bit spread over a word, the
// ballot, and one three-input operation m & ~(ballot ^ bit) per half (nine as
// the plain expression compiles).
__device__ __forceinline__ uint64_t digit_peers(uint32_t d, bool act) {
    const uint64_t m = ballot(act);
    uint32_t lo = (uint32_t)m, hi = (uint32_t)(m >> 32);
#pragma unroll
    for (int b = 0; b < kRadixBits; ++b) {
        const uint32_t bit = (uint32_t)((int32_t)(d << (31 - b)) >> 31);
        const uint64_t bal = ballot(bit != 0u);
        lo = __builtin_amdgcn_bitop3_b32(lo, (uint32_t)bal, bit, 0x90);
        hi = __builtin_amdgcn_bitop3_b32(hi, (uint32_t)(bal >> 32), bit, 0x90);
    }
    return ((uint64_t)hi << 32) | lo;
}

}  // namespace gv

// ======================================================================
// Primitives with decoupled look-back between workgroups.  Look-back status
// words live in a caller-provided region that must be zero before the launch
// (the batch pipeline clears it in its first kernel).  Every wait is bounded:
// a wait that runs out sets an error flag instead of hanging, and the callers
// treat the result as failed.
// ======================================================================
namespace gv {

constexpr uint32_t kSpinLimit = kSpinLimitDefault;

constexpr int kScan1Items = 8;

// Status words carry their own value (flag and count in one word), so no other
// data is ordered by them: relaxed loads and stores at device scope suffice.
__device__ __forceinline__ uint32_t ld_status32(uint32_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_status32(uint32_t* p, uint32_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---------------------------------------------------------------- scan2
// Two-kernel exclusive scan without inter-tile waits: the first kernel
// reduces each tile, the second recomputes its tile prefix by reducing the
// partials of all earlier tiles (up to kScan2MaxTiles, read from L2; with
// more tiles a one-workgroup kernel between the two scans the partials) and
// scans its tile.  Inputs are evaluated twice, outputs written once.  On a
// context with a scan state (the graph's stream), inputs of 2 to
// kChainTiles tiles take a one-kernel form instead (k_scan2_chain below).
//
// The source is a gather: it splits each element into its memory reads and
// the arithmetic on them, so that a thread issues the reads of all of its
// elements before it waits on any of them.
//   uint64_t limit(uint64_t n)          live elements (<= n, may be read from
//                                       device memory); the rest count 0
//   Rec load(uint64_t i, bool ok)       first-level reads of element i (always
//                                       i < n); every address must be valid
//                                       also when !ok, and no read may sit
//                                       behind a branch
//   void deref(Rec&)                    reads at addresses that load() read
//                                       (same rules)
//   ull value(uint64_t i, const Rec&)   the element's value (called when ok)
// The sink takes (i, rec, lim, exclusive prefix) for every i < n; the
// element is live when i < lim.  A sink may also define
//   void finish()                       run by the first wave of the last
//                                       workgroup once the total is written
// A thread takes kScan1Items elements.
template <typename Out, typename = void>
struct scan2_has_finish : std::false_type {};
template <typename Out>
struct scan2_has_finish<Out, std::void_t<decltype(std::declval<const Out&>().finish())>>
    : std::true_type {};

template <typename In>
__global__ __launch_bounds__(kThreads) void k_scan2_reduce(In in, uint64_t n,
                                                           unsigned long long* part) {
    constexpr int kI = kScan1Items;
    __shared__ unsigned long long s_w[kWaves];
    const uint64_t lim = in.limit(n);
    const uint64_t base = (uint64_t)blockIdx.x * kThreads * kI + threadIdx.x;
    typename In::Rec r[kI];
#pragma unroll
    for (int j = 0; j < kI; ++j) {
        const uint64_t i = base + (uint64_t)j * kThreads;
        r[j] = in.load(i < n ? i : n - 1, i < lim);
    }
#pragma unroll
    for (int j = 0; j < kI; ++j) in.deref(r[j]);
    unsigned long long s = 0;
#pragma unroll
    for (int j = 0; j < kI; ++j) {
        const uint64_t i = base + (uint64_t)j * kThreads;
        s += i < lim ? in.value(i, r[j]) : 0ull;
    }
    s = block_sum(s, s_w);
    if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// Exclusive scan of the nt tile sums in place (one workgroup), for inputs
// with more tiles than the apply kernel adds up itself.  A serial chain of
// rounds: 1024 threads take 8 sums each per round, so 4900 tiles (10^7
// elements) are one round of 6 us (256 threads with one sum each took 46).
constexpr int kPartThreads = 1024, kPartItems = 8;
static __global__ __launch_bounds__(kPartThreads) void k_scan2_partials(unsigned long long* part,
                                                                        uint64_t nt) {
    __shared__ unsigned long long lds[kPartThreads / 64];
    unsigned long long carry = 0;
    const int w = threadIdx.x >> 6;
    for (uint64_t b = 0; b < nt; b += (uint64_t)kPartThreads * kPartItems) {
        const uint64_t i0 = b + (uint64_t)threadIdx.x * kPartItems;
        unsigned long long x[kPartItems], sum = 0;
#pragma unroll
        for (int j = 0; j < kPartItems; ++j) x[j] = part[i0 + j < nt ? i0 + j : nt - 1];
#pragma unroll
        for (int j = 0; j < kPartItems; ++j) {
            x[j] = i0 + j < nt ? x[j] : 0ull;
            sum += x[j];
        }
        const unsigned long long inc = wave_incl_scan(sum);
        if (lane_id() == 63) lds[w] = inc;
        __syncthreads();
        unsigned long long run = carry + inc - sum;
#pragma unroll
        for (int k = 0; k < kPartThreads / 64; ++k) {
            const unsigned long long v = lds[k];
            run += k < w ? v : 0ull;
            carry += v;
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kPartItems; ++j) {
            if (i0 + j < nt) part[i0 + j] = run;
            run += x[j];
        }
    }
}

// scanned: part already holds exclusive tile prefixes
template <typename In, typename Out>
__global__ __launch_bounds__(kThreads) void k_scan2_apply(In in, Out out, uint64_t n,
                                                          const unsigned long long* part,
                                                          int scanned,
                                                          unsigned long long* total) {
    constexpr int kI = kScan1Items;
    __shared__ unsigned long long s_w[kI][kWaves];
    __shared__ unsigned long long s_p[kWaves];
    const uint64_t lim = in.limit(n);
    const uint64_t base = (uint64_t)blockIdx.x * kThreads * kI + threadIdx.x;
    typename In::Rec r[kI];
#pragma unroll
    for (int j = 0; j < kI; ++j) {
        const uint64_t i = base + (uint64_t)j * kThreads;
        r[j] = in.load(i < n ? i : n - 1, i < lim);
    }
#pragma unroll
    for (int j = 0; j < kI; ++j) in.deref(r[j]);
    unsigned long long p = 0;
    if (scanned) {
        p = threadIdx.x == 0 ? part[blockIdx.x] : 0ull;
    } else {
        for (uint32_t t = threadIdx.x; t < blockIdx.x; t += kThreads) p += part[t];
    }
    // one wave scan per row of the tile, then a single exchange of the
    // per-wave row totals
    unsigned long long x[kI], inc[kI];
#pragma unroll
    for (int j = 0; j < kI; ++j) {
        const uint64_t i = base + (uint64_t)j * kThreads;
        x[j] = i < lim ? in.value(i, r[j]) : 0ull;
        inc[j] = wave_incl_scan(x[j]);
    }
    const int w = threadIdx.x >> 6;
    if (lane_id() == 63) {
#pragma unroll
        for (int j = 0; j < kI; ++j) s_w[j][w] = inc[j];
    }
    unsigned long long run = block_sum(p, s_p);  // its barriers publish s_w
#pragma unroll
    for (int j = 0; j < kI; ++j) {
        const uint64_t i = base + (uint64_t)j * kThreads;
        unsigned long long before = 0, tot = 0;
#pragma unroll
        for (int q = 0; q < kWaves; ++q) {
            const unsigned long long v = s_w[j][q];
            before += q < w ? v : 0ull;
            tot += v;
        }
        if (i < n) out(i, r[j], lim, run + before + inc[j] - x[j]);
        run += tot;
    }
    if (total && blockIdx.x == gridDim.x - 1 && threadIdx.x == kThreads - 1) *total = run;
    if constexpr (scan2_has_finish<Out>::value) {
        // a sink may finish the scan in its last workgroup: the first wave
        // runs out.finish() once the total is written
        if (blockIdx.x == gridDim.x - 1) {
            __syncthreads();
            if (threadIdx.x < 64) out.finish();
        }
    }
}

// One-kernel form for inputs of 2 to kChainTiles tiles: a workgroup takes
// its tile by ticket (so every tile it waits for belongs to a workgroup that
// started before it), publishes the tile's sum (plus one: zero is unset), adds
// the sums of all earlier tiles (each thread a strided share of them,
// bounded waits on relaxed loads of words that carry their own value), and
// scans its tile as the apply kernel does.  A tile waits
// for the earlier tiles' own sums, not their prefixes, so the waits do not
// chain.  The last workgroup to finish returns the state to zero.
template <typename In, typename Out>
__global__ __launch_bounds__(kThreads) void k_scan2_chain(In in, Out out, uint64_t n,
                                                          uint32_t nt, ChainState* st,
                                                          uint32_t* err,
                                                          unsigned long long* total) {
    constexpr int kI = kScan1Items;
    __shared__ unsigned long long s_w[kI][kWaves];
    __shared__ unsigned long long s_p[kWaves];
    __shared__ uint32_t s_tile, s_last;
    if (threadIdx.x == 0) s_tile = atomicAdd(&st->ticket, 1u);
    __syncthreads();
    const uint32_t tile = s_tile;
    const uint64_t lim = in.limit(n);
    const uint64_t base = (uint64_t)tile * kThreads * kI + threadIdx.x;
    typename In::Rec r[kI];
#pragma unroll
    for (int j = 0; j < kI; ++j) {
        const uint64_t i = base + (uint64_t)j * kThreads;
        r[j] = in.load(i < n ? i : n - 1, i < lim);
    }
#pragma unroll
    for (int j = 0; j < kI; ++j) in.deref(r[j]);
    unsigned long long x[kI], inc[kI];
#pragma unroll
    for (int j = 0; j < kI; ++j) {
        const uint64_t i = base + (uint64_t)j * kThreads;
        x[j] = i < lim ? in.value(i, r[j]) : 0ull;
        inc[j] = wave_incl_scan(x[j]);
    }
    const int w = threadIdx.x >> 6;
    if (lane_id() == 63) {
#pragma unroll
        for (int j = 0; j < kI; ++j) s_w[j][w] = inc[j];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long t = 0;
#pragma unroll
        for (int j = 0; j < kI; ++j)
#pragma unroll
            for (int q = 0; q < kWaves; ++q) t += s_w[j][q];
        __hip_atomic_store(&st->sum[tile], t + 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    unsigned long long p = 0;
    for (uint32_t k = threadIdx.x; k < tile; k += kThreads) {
        uint32_t spins = 0;
        unsigned long long x;
        while ((x = __hip_atomic_load(&st->sum[k], __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_AGENT)) == 0ull) {
            if (++spins >= kSpinLimit) {
                atomicOr(err, 1u);
                x = 1ull;
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
        p += x - 1ull;
    }
    unsigned long long run = block_sum(p, s_p);
#pragma unroll
    for (int j = 0; j < kI; ++j) {
        const uint64_t i = base + (uint64_t)j * kThreads;
        unsigned long long before = 0, tot = 0;
#pragma unroll
        for (int q = 0; q < kWaves; ++q) {
            const unsigned long long v = s_w[j][q];
            before += q < w ? v : 0ull;
            tot += v;
        }
        if (i < n) out(i, r[j], lim, run + before + inc[j] - x[j]);
        run += tot;
    }
    const bool last = tile == nt - 1;
    if (total && last && threadIdx.x == kThreads - 1) *total = run;
    __syncthreads();
    if constexpr (scan2_has_finish<Out>::value) {
        if (last && threadIdx.x < 64) out.finish();
    }
    if (threadIdx.x == 0) s_last = atomicAdd(&st->done, 1u) == nt - 1 ? 1u : 0u;
    __syncthreads();
    if (s_last) {
        // every workgroup has read what it waits for
        for (uint32_t t = threadIdx.x; t < nt; t += kThreads) st->sum[t] = 0ull;
        if (threadIdx.x == 0) {
            st->ticket = 0u;
            st->done = 0u;
        }
    }
}

// tiles the apply kernel adds up itself; beyond, a middle kernel scans them
constexpr uint64_t kScan2MaxTiles = 2048;
// partial words any scan2 over n elements needs
inline uint64_t scan2_parts(uint64_t n) {
    return div_up(std::max<uint64_t>(n, 1), (uint64_t)kThreads * kScan1Items);
}

// tiles of a scan2 over n elements (one tile: no reduce kernel)
inline uint64_t scan2_tiles(uint64_t n) { return div_up(n, (uint64_t)kThreads * kScan1Items); }

// Exclusive scan of in(i), i < n, as out(i, rec, lim, prefix); total ->
// *total.  `part` holds scan2_parts(n) words.
template <typename In, typename Out>
void scan2(Ctx& c, const char* name, In in, Out out, uint64_t n, unsigned long long* part,
           unsigned long long* total) {
    if (n == 0) return;
    const uint64_t nt = scan2_tiles(n);
    if (nt > 0xffffffffull) fail(GV_EINVAL, "scan too large");
    if (nt > 1 && nt <= kChainTiles && c.chain) {
        c.launch(name, k_scan2_chain<In, Out>, nt, kThreads, in, out, n, (uint32_t)nt,
                 (ChainState*)c.chain, c.chain_err, total);
        return;
    }
    // a single tile adds no earlier partials: the apply kernel is the scan
    if (nt > 1) c.launch(name, k_scan2_reduce<In>, nt, kThreads, in, n, part);
    const int scanned = nt > kScan2MaxTiles ? 1 : 0;
    if (scanned) c.launch(name, k_scan2_partials, 1, kPartThreads, part, nt);
    c.launch(name, k_scan2_apply<In, Out>, nt, kThreads, in, out, n,
             (const unsigned long long*)part, scanned, total);
}

// ---------------------------------------------------------------- onesweep
// Stable LSD radix sort: one histogram kernel for every pass, then one kernel
// per 8-bit digit pass (k_os_pass).  The number of keys may live on the device
// (n_dev); grids are sized for n_max.
#ifndef GV_OS_ITEMS
#define GV_OS_ITEMS 16
#endif
constexpr int kOsItems = GV_OS_ITEMS;  // keys per tile = kThreads * kOsItems
constexpr uint64_t kOsTile = (uint64_t)kThreads * kOsItems;  // 4096
constexpr uint32_t kOsAgg = 1u << 30, kOsIncl = 2u << 30, kOsMask = (1u << 30) - 1;

inline int os_passes(int bits) { return (bits + kRadixBits - 1) / kRadixBits; }
// Digit histograms: every histogram workgroup writes its own counts (no
// atomics), one small kernel adds them up.  A workgroup takes a key per thread
// and turn, two workgroups a compute unit: with four keys per thread 10^5 pairs
// filled 25 units (pack 13.8 us, now 6.8), 10^6 pairs one workgroup a unit (21.7,
// now 16.7; building from 1.7 * 10^7 88 -> 69); 10^7 pairs take 109 us either
// way.
constexpr uint64_t kHistGroups = 512;
constexpr uint64_t kHistTile = 1024;
inline uint64_t os_hist_groups(uint64_t n) {
    return std::min<uint64_t>(div_up(std::max<uint64_t>(n, 1), kHistTile), kHistGroups);
}
// uint32 words of state a sort needs: tile counters and look-back status
// (the first os_zero_words, which must be zeroed), then the histograms and
// the per-group histograms.
// The pass kernel's own tiles, and its three-level prefix: a group is kOsGroup
// tiles, a super group kOsGroup groups.
// Keys per thread of a pass: 8 up to kPsLong keys, then 16, whose longer runs
// (32 keys a digit on average) and half as many tiles cost less per key once
// the device is full many times over: 10^6 keys 14.7 us a pass against 18.4,
// 10^7 keys 66.1 against 58.5, 1.7 * 10^7 keys 104 against 89.
constexpr int kPsThreads = 512, kPsWaves = kPsThreads / 64;
constexpr int kPsRounds = 8, kPsRoundsLong = 16, kPsRoundsShort = 4;
constexpr uint64_t kOsGroup = 16;
constexpr uint64_t kPsLong = 1ull << 22, kPsShort = 1ull << 18;
// (Below a tile per compute unit, shorter tiles give more of them and a
// shorter chain each: 10^5 keys 8.4 us a pass against 7.9, with values 9.3
// against 7.8, 10^6 keys 17.0 against 21.0; two keys per thread 8.5 and 8.2.
// With values the longest tile's LDS would leave one workgroup per unit.)
inline int ps_rounds(uint64_t n, bool vals) {
    return n <= kPsShort ? kPsRoundsShort : n > kPsLong && !vals ? kPsRoundsLong : kPsRounds;
}
inline uint64_t ps_tiles(uint64_t n, bool vals) {
    return div_up(std::max<uint64_t>(n, 1), (uint64_t)kPsThreads * ps_rounds(n, vals));
}
// status words per digit and pass: tiles, groups, super groups
inline uint64_t ps_status(uint64_t n, bool vals) {
    const uint64_t t = ps_tiles(n, vals), g = div_up(t, kOsGroup);
    return t + g + div_up(g, kOsGroup);
}
// (vals: the sort carries values)
inline uint64_t os_zero_words(uint64_t n_max, int bits, bool vals = false) {
    return 64 + (uint64_t)os_passes(bits) * ps_status(n_max, vals) * kRadix;
}
inline uint64_t os_words(uint64_t n_max, int bits, bool vals = false) {
    const uint64_t p = (uint64_t)os_passes(bits);
    return os_zero_words(n_max, bits, vals) + p * kRadix + os_hist_groups(n_max) * p * kRadix;
}

constexpr int kOsThreads = 1024;
static_assert(kHistTile == kOsThreads, "a key per thread");
constexpr int kOsWaves = kOsThreads / 64;
static_assert(kOsThreads == 4 * kRadix, "the pass kernel works in four quarters of 256 threads");
constexpr int kOsRounds = (int)(kOsTile / kOsThreads);  // keys per thread
// exclusive scan across a kOsThreads workgroup (all threads call it)
__device__ __forceinline__ uint32_t os_block_scan(uint32_t x, uint32_t* lds, uint32_t& total) {
    uint32_t inc = wave_incl_scan(x);
    const int w = threadIdx.x >> 6;
    if (lane_id() == 63) lds[w] = inc;
    __syncthreads();
    uint32_t off = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < kOsWaves; ++i) {
        const uint32_t v = lds[i];
        off += (i < w) ? v : 0u;
        tot += v;
    }
    __syncthreads();
    total = tot;
    return off + inc - x;
}

// LDS of the one-tile sort below.
struct TileSortLds {
    uint16_t cnt[kOsRounds * kOsWaves][kRadix];
    uint32_t part[4][kRadix];
    uint32_t start[kRadix];
    uint32_t w[kOsWaves];
    uint64_t skey[kOsTile];
};

// Tiles of at most kTileBitonicMax keys are sorted by a bitonic network in
// LDS, in log2(m) (log2(m) + 1) / 2 compare-exchange steps for m keys padded
// to a power of two with all-ones keys, instead of five barriers per radix
// pass.  The network is not stable, but every caller's keys are whole
// records (an edge key, a destination, or a key with its input position in
// the low bits), so keys that compare equal are identical and the result is
// the array a stable sort gives.
constexpr uint64_t kTileBitonicMax = 2048;

__device__ __forceinline__ void tile_bitonic(uint64_t (&key)[kOsRounds], uint32_t n,
                                             uint64_t sentinel, TileSortLds& L) {
    static_assert(kTileBitonicMax <= kOsTile, "the network works in the tile's LDS");
    const uint32_t t = threadIdx.x;
    uint32_t m = 2;
    while (m < n) m <<= 1;
#pragma unroll
    for (int j = 0; j < kOsRounds; ++j) {
        const uint32_t i = (uint32_t)j * kOsThreads + t;
        if (i < m) L.skey[i] = i < n ? key[j] : ~0ull;
    }
    // Thread c compares the pair (i, i + h), i being c with a zero bit
    // inserted at h.  While h <= 64 the pairs of a wave lie in its own 128
    // elements, so a step needs the whole workgroup's barrier only when it or
    // the step before it has h >= 128; else the wave's own order suffices.
    static_assert(kTileBitonicMax / 2 <= kOsThreads, "one pair per thread");
    uint32_t hprev = m;  // the loads above cross waves
    for (uint32_t k = 2; k <= m; k <<= 1) {
        for (uint32_t h = k >> 1; h > 0; h >>= 1) {
            if (h >= 128 || hprev >= 128) {
                __syncthreads();
            } else {
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            }
            hprev = h;
            if (t < m / 2) {
                const uint32_t i = ((t & ~(h - 1)) << 1) | (t & (h - 1));
                const uint32_t p = i + h;
                const uint64_t a = L.skey[i], b = L.skey[p];
                if ((a > b) == ((i & k) == 0)) {
                    L.skey[i] = b;
                    L.skey[p] = a;
                }
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kOsRounds; ++j) {
        const uint32_t i = (uint32_t)j * kOsThreads + t;
        key[j] = i < n ? L.skey[i] : sentinel;
    }
    __syncthreads();  // the caller may reuse the LDS
}

// Stable LSD sort of one tile in LDS: thread t holds key[j] = element
// j * kOsThreads + t, the first n live; `passes` 8-bit digits (the ranking of
// the pass kernel on a single tile, so no look-back).  key[] comes back
// holding the sorted order in the same layout, `sentinel` past n.  Every
// thread of the workgroup calls it (barriers inside).  Live keys must be
// below 2^(8 * passes).
__device__ __forceinline__ void tile_sort(uint64_t (&key)[kOsRounds], uint64_t n, int passes,
                                          uint64_t sentinel, TileSortLds& L) {
    if (n <= kTileBitonicMax) {
        if (n > 1) {
            tile_bitonic(key, (uint32_t)n, sentinel, L);
        } else {
            // nothing to order: element 0 stays where it is
            if (threadIdx.x >= n) key[0] = sentinel;
#pragma unroll
            for (int j = 1; j < kOsRounds; ++j) key[j] = sentinel;
        }
        return;
    }
    const uint32_t t = threadIdx.x;
    const int w = t >> 6;
    const uint32_t d = t & (kRadix - 1), q = t >> 8;
    constexpr int kQRows = kOsRounds * kOsWaves / 4;
    for (int p = 0; p < passes; ++p) {
        const int shift = p * kRadixBits;
        {
            uint32_t* c32 = (uint32_t*)&L.cnt[0][0];
            for (int i = t; i < kOsRounds * kOsWaves * kRadix / 2; i += kOsThreads) c32[i] = 0;
        }
        __syncthreads();
        uint16_t rk[kOsRounds];
#pragma unroll
        for (int j = 0; j < kOsRounds; ++j) {
            const bool act = (uint64_t)j * kOsThreads + t < n;
            const uint32_t dg = (uint32_t)(key[j] >> shift) & (kRadix - 1);
            const uint64_t peers = digit_peers(dg, act);
            rk[j] = (uint16_t)rank_below(peers);
            if (act && rk[j] == 0) L.cnt[j * kOsWaves + w][dg] = (uint16_t)popc64(peers);
        }
        __syncthreads();
        // rows in key order: exclusive prefixes per digit, 16 rows per quarter
        uint32_t run = 0;
#pragma unroll
        for (int r = 0; r < kQRows; ++r) {
            const uint32_t c = L.cnt[q * kQRows + r][d];
            L.cnt[q * kQRows + r][d] = (uint16_t)run;
            run += c;
        }
        L.part[q][d] = run;
        __syncthreads();
        uint32_t qoff = 0;
        for (uint32_t qq = 0; qq < q; ++qq) qoff += L.part[qq][d];
        if (qoff) {
#pragma unroll
            for (int r = 0; r < kQRows; ++r) L.cnt[q * kQRows + r][d] += (uint16_t)qoff;
        }
        const uint32_t dcount = L.part[0][d] + L.part[1][d] + L.part[2][d] + L.part[3][d];
        uint32_t tot;
        const uint32_t ex = os_block_scan(q == 0 ? dcount : 0u, L.w, tot);
        if (q == 0) L.start[d] = ex;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kOsRounds; ++j) {
            if ((uint64_t)j * kOsThreads + t < n) {
                const uint32_t dg = (uint32_t)(key[j] >> shift) & (kRadix - 1);
                L.skey[L.start[dg] + L.cnt[j * kOsWaves + w][dg] + rk[j]] = key[j];
            }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kOsRounds; ++j) {
            const uint64_t i = (uint64_t)j * kOsThreads + t;
            key[j] = i < n ? L.skey[i] : sentinel;
        }
        __syncthreads();  // skey and cnt are rewritten by the next pass
    }
}

// Histogram counting: 0 = the lowest lane of each group of equal digits adds
// the group's size (eight ballots per digit, no conflicting LDS atomics);
// 1 = every lane adds one to a histogram shared by a quarter of the
// workgroup (LDS atomics, conflicts only between equal digits).
#ifndef GV_OS_HIST_MODE
#define GV_OS_HIST_MODE 1
#endif
#ifndef GV_OS_HIST_COPIES
#define GV_OS_HIST_COPIES 4
#endif
constexpr int kOsHistMode = GV_OS_HIST_MODE;
constexpr int kOsHistCopies = kOsHistMode == 1 ? GV_OS_HIST_COPIES : 1;

template <typename K>
__global__ __launch_bounds__(kOsThreads) void k_os_hist(const K* keys, const uint32_t* n_dev,
                                                        uint64_t n_max, int passes,
                                                        uint32_t* hpart, uint32_t* state,
                                                        uint64_t state_words, uint32_t* clear,
                                                        uint32_t clear_words) {
    __shared__ uint32_t h[kOsHistCopies][8][kRadix];
    const uint64_t nt = (uint64_t)gridDim.x * kOsThreads;
    const uint64_t me = (uint64_t)blockIdx.x * kOsThreads + threadIdx.x;
    for (uint64_t i = me; i < state_words; i += nt) state[i] = 0;
    for (uint64_t i = me; i < clear_words; i += nt) clear[i] = 0;
    const uint64_t n = n_dev ? min<uint64_t>(*n_dev, n_max) : n_max;
    for (int i = threadIdx.x; i < kOsHistCopies * 8 * kRadix; i += kOsThreads)
        (&h[0][0][0])[i] = 0;
    __syncthreads();
    const uint32_t copy = kOsHistCopies == 1 ? 0u : (threadIdx.x >> 6) & (kOsHistCopies - 1);
    // tiles of n_max: loads need not wait for n, counting masks with it
    const uint64_t ntiles = (n_max + kHistTile - 1) / kHistTile;
    for (uint64_t tl = blockIdx.x; tl < ntiles; tl += gridDim.x) {
        const uint64_t i = tl * kHistTile + threadIdx.x;
        const K k = i < n_max ? keys[i] : K(0);
        const bool act = i < n;
        for (int p = 0; p < passes; ++p) {
            const uint32_t d = (uint32_t)(k >> (p * kRadixBits)) & (kRadix - 1);
            if (kOsHistMode == 1) {
                if (act) atomicAdd(&h[copy][p][d], 1u);
            } else {
                const uint64_t peers = digit_peers(d, act);
                if (act && rank_below(peers) == 0) atomicAdd(&h[0][p][d], popc64(peers));
            }
        }
    }
    __syncthreads();
    uint32_t* out = hpart + (uint64_t)blockIdx.x * passes * kRadix;
    for (int i = threadIdx.x; i < passes * kRadix; i += kOsThreads) {
        uint32_t x = 0;
#pragma unroll
        for (int c = 0; c < kOsHistCopies; ++c) x += h[c][i / kRadix][i % kRadix];
        out[i] = x;
    }
}

// hist[i] = sum over the histogram workgroups of their count i: a
// workgroup takes 16 counters, its 16 row groups each add every 16th
// workgroup's count with independent loads, LDS adds the row groups
// (when vpart is given, workgroup 0 also adds the groups' vpart counts into
// *vtotal, and their kpart sums into *ktotal)
static __global__ __launch_bounds__(kThreads) void k_os_hist_sum(
    const uint32_t* hpart, uint32_t groups, uint32_t words, uint32_t* hist, const uint32_t* vpart,
    unsigned long long* vtotal, const unsigned long long* kpart, unsigned long long* ktotal) {
    __shared__ uint32_t red[16][17];
    __shared__ unsigned long long s_v[kWaves];
    if (vpart && blockIdx.x == 0) {
        unsigned long long x = 0, y = 0;
        for (uint32_t i = threadIdx.x; i < groups; i += kThreads) {
            x += vpart[i];
            y += kpart[i];
        }
        const unsigned long long t = block_sum(x, s_v);
        const unsigned long long u = block_sum(y, s_v);
        if (threadIdx.x == 0) {
            *vtotal = t;
            *ktotal = u;
        }
    }
    if (words == 0) return;
    const uint32_t col = threadIdx.x & 15, rg = threadIdx.x >> 4;
    const uint32_t i = blockIdx.x * 16 + col;
    const uint32_t ic = i < words ? i : 0u;
    uint32_t s = 0;
    constexpr uint32_t kRows = (uint32_t)(kHistGroups / 16);
#pragma unroll
    for (uint32_t r = 0; r < kRows; ++r) {
        const uint32_t gi = rg + 16 * r;
        const uint32_t x = hpart[(uint64_t)(gi < groups ? gi : 0u) * words + ic];
        s += gi < groups ? x : 0u;
    }
    red[rg][col] = s;
    __syncthreads();
    if (rg == 0 && i < words) {
        uint32_t t = 0;
#pragma unroll
        for (int k = 0; k < 16; ++k) t += red[k][col];
        hist[i] = t;
    }
}

// One pass over 8 bits at `shift`.  A wave ranks its keys by itself: for each
// row of 64, eight ballots find the lanes with the same digit, the wave's own
// counter of the digit (LDS) gives the keys before the row, and the row's
// first lane advances it, so ranking takes no barrier.  The tile's counts are
// published, its keys placed in digit order in LDS, and only then are the
// counts of earlier tiles gathered: the earlier tiles of the tile's group, the
// earlier groups of its super group, and the super groups before it back to
// the first whose inclusive prefix stands, all loads issued together (two
// lanes per digit, eight words each per level).  The group's last tile
// publishes the group's counts, the super group's last tile its counts and
// its inclusive prefix.  Each digit's run is then written with consecutive
// lanes.
//
// Bound: at 245 tiles (10^6 keys) the chain of dependent phases, from a few
// thousand tiles on issue and the scattered writes (runs of 16 or 32 keys).  A
// first form ranked with nine vector instructions per digit bit and a row of
// LDS counters per 64 keys, and looked back before it placed its keys: 10^6
// keys 16.9 us a pass, now 14.7; 10^7 keys 88 (1.8 TB/s), now 58 (2.7 TB/s).
template <typename K, bool HasVal, int kRounds>
__global__ __launch_bounds__(kPsThreads) void k_os_pass(const K* kin, K* kout, const uint32_t* vin,
                                                        uint32_t* vout, const uint32_t* n_dev,
                                                        uint64_t n_max, int shift,
                                                        const uint32_t* hist, uint32_t* status,
                                                        uint32_t* counter, int block_tiles,
                                                        uint32_t* err, uint32_t spin_limit) {
    static_assert(kPsThreads == 2 * kRadix, "two lanes per digit look back");
    constexpr uint32_t kL = (uint32_t)kOsGroup / 2;  // words per lane and level
    constexpr uint64_t kPsTile = (uint64_t)kPsThreads * kRounds;
    constexpr uint32_t kWaveKeys = 64 * kRounds;
    __shared__ uint16_t cnt[kPsWaves][kRadix];  // counts, then exclusive prefixes over the waves
    __shared__ K skey[kPsTile];
    __shared__ uint32_t sval[HasVal ? kPsTile : 1];
    __shared__ uint32_t s_lstart[kRadix];  // start of the digit's run inside the tile
    __shared__ uint32_t s_count[kRadix];   // its length
    __shared__ uint32_t s_off[kRadix];     // its global start minus s_lstart
    __shared__ unsigned long long s_w[kPsWaves];
    __shared__ uint32_t s_tile;
    const uint32_t t = threadIdx.x, w = t >> 6, lane = lane_id();
    // the pass histogram and the key count do not depend on the tile
    const uint32_t hv = t < kRadix ? hist[t] : 0u;
    const uint64_t n = n_dev ? min<uint64_t>(*n_dev, n_max) : n_max;
    // Tile ids: when every tile's workgroup fits on the device at once, the
    // workgroup index (all tiles run together, so each one a tile waits for
    // is running); else a ticket in launch order, so that every tile a tile
    // waits for has started.
    uint64_t tile = blockIdx.x;
    if (!block_tiles) {
        if (t == 0) s_tile = atomicAdd(counter, 1u);
        __syncthreads();
        tile = s_tile;
    }
    const uint64_t base = tile * kPsTile;
    const uint64_t mine = base + (uint64_t)w * kWaveKeys + lane;
    // (a digit is a byte of the key: it lies in one half of it)
    const int half = shift & 31;
    auto digit = [&](K k) {
        const uint32_t x = shift < 32 ? (uint32_t)k : (uint32_t)((uint64_t)k >> 32);
        return (x >> half) & (kRadix - 1);
    };
    K key[kRounds];
    uint32_t val[kRounds];
    // loads bounded by n_max (the buffer size), so they need not wait for n
#pragma unroll
    for (int j = 0; j < kRounds; ++j) {
        const uint64_t i = mine + 64 * j;
        const bool in = i < n_max;
        key[j] = in ? kin[i] : K(0);
        if (HasVal) val[j] = in ? vin[i] : 0u;
    }
#pragma unroll
    for (int i = 0; i < kRadix / 64; ++i) cnt[w][i * 64 + lane] = 0;
    uint32_t rk[kRounds];
    wave_fence();
#pragma unroll
    for (int j = 0; j < kRounds; ++j) {
        const bool act = mine + 64 * j < n;
        const uint32_t d = digit(key[j]);
        const uint64_t peers = digit_peers(d, act);
        const uint32_t r = rank_below(peers);
        const uint32_t before = cnt[w][d];
        wave_fence();
        if (act && r == 0) cnt[w][d] = (uint16_t)(before + popc64(peers));
        wave_fence();
        rk[j] = before + r;
    }
    __syncthreads();
    uint32_t dcount = 0;
    if (t < kRadix) {
        uint32_t c[kPsWaves];
#pragma unroll
        for (int q = 0; q < kPsWaves; ++q) c[q] = cnt[q][t];
#pragma unroll
        for (int q = 0; q < kPsWaves; ++q) {
            cnt[q][t] = (uint16_t)dcount;
            dcount += c[q];
        }
        st_status32(status + tile * kRadix + t, kOsAgg | dcount);
    }
    // global start of each digit (pass histogram) and start inside the tile:
    // one scan of both, the histogram in the high half (neither half carries)
    {
        const unsigned long long x = ((unsigned long long)hv << 32) | dcount;
        const unsigned long long inc = wave_incl_scan(x);
        if (lane == 63) s_w[w] = inc;
        __syncthreads();
        if (t < kRadix) {
            unsigned long long ex = inc - x;
            for (uint32_t i = 0; i < w; ++i) ex += s_w[i];
            s_lstart[t] = (uint32_t)ex;
            s_count[t] = dcount;
            s_off[t] = (uint32_t)(ex >> 32) - (uint32_t)ex;
        }
    }
    __syncthreads();
    // place keys in tile order of their digit
#pragma unroll
    for (int j = 0; j < kRounds; ++j) {
        if (mine + 64 * j < n) {
            const uint32_t d = digit(key[j]);
            const uint32_t lp = s_lstart[d] + cnt[w][d] + rk[j];
            skey[lp] = key[j];
            if (HasVal) sval[lp] = val[j];
        }
    }
    {
        // (32-bit places: a pass has fewer than 2^30 / kPsTile tiles)
        const uint32_t tl = (uint32_t)tile, nt = gridDim.x;
        const uint32_t ld = t >> 1, lq = t & 1, q8 = lq * kL;
        const uint32_t G = tl / (uint32_t)kOsGroup, S = G / (uint32_t)kOsGroup;
        const uint32_t g0 = G * (uint32_t)kOsGroup, s0 = S * (uint32_t)kOsGroup;
        uint32_t* tst = status + ld;
        uint32_t* gst = tst + (uint64_t)nt * kRadix;
        // waits for one word, which is polled again until it is set
        auto settle = [&](uint32_t x, uint32_t* p, bool real) {
            if (real && ((x >> 30) == 0 || spin_limit == 0)) {
                uint32_t spins = 0;
                while ((x >> 30) == 0 && spins++ < spin_limit) x = ld_status32(p);
                if ((x >> 30) == 0 || spin_limit == 0) {
                    *err = 1;
                    x = kOsIncl;
                }
            }
            return x;
        };
        uint32_t a[kL], b[kL];
#pragma unroll
        for (uint32_t k = 0; k < kL; ++k)
            a[k] = g0 + q8 + k < tl ? ld_status32(tst + (uint64_t)(g0 + q8 + k) * kRadix) : kOsAgg;
#pragma unroll
        for (uint32_t k = 0; k < kL; ++k)
            b[k] = s0 + q8 + k < G ? ld_status32(gst + (uint64_t)(s0 + q8 + k) * kRadix) : kOsAgg;
        uint32_t local = 0, groups = 0;
#pragma unroll
        for (uint32_t k = 0; k < kL; ++k)
            local += settle(a[k], tst + (uint64_t)(g0 + q8 + k) * kRadix, g0 + q8 + k < tl) &
                     kOsMask;
        local += pair_read(local);
        const uint32_t own = s_count[ld];
        if (tl - g0 == kOsGroup - 1 && lq == 0)
            st_status32(gst + (uint64_t)G * kRadix, kOsAgg | (local + own));
#pragma unroll
        for (uint32_t k = 0; k < kL; ++k)
            groups += settle(b[k], gst + (uint64_t)(s0 + q8 + k) * kRadix, s0 + q8 + k < G) &
                      kOsMask;
        groups += pair_read(groups);
        uint32_t prefix = local + groups;
        uint32_t* sst = gst + (uint64_t)((nt + kOsGroup - 1) / kOsGroup) * kRadix;
        const bool last = tl % (kOsGroup * kOsGroup) == kOsGroup * kOsGroup - 1;
        if (S > 0) {  // uniform over the workgroup
            if (last && lq == 0) st_status32(sst + (uint64_t)S * kRadix, kOsAgg | (prefix + own));
            for (uint32_t s1 = S;; s1 -= (uint32_t)kOsGroup) {
                // super groups s1 - 1, s1 - 2, ...: this lane's eight, newest
                // first; before the first stands an inclusive zero
                uint32_t sum = 0;
                bool incl = false;
#pragma unroll
                for (uint32_t k = 0; k < kL; ++k)
                    a[k] = q8 + k < s1 ? ld_status32(sst + (uint64_t)(s1 - 1 - q8 - k) * kRadix)
                                       : kOsIncl;
#pragma unroll
                for (uint32_t k = 0; k < kL; ++k) {
                    if (!incl) {
                        const uint32_t x =
                            settle(a[k], sst + (uint64_t)(s1 - 1 - q8 - k) * kRadix, q8 + k < s1);
                        sum += x & kOsMask;
                        incl = (x >> 30) == 2;
                    }
                }
                const uint32_t osum = pair_read(sum);
                const bool oincl = pair_read(incl) != 0;
                // the first lane's words are the newer ones
                const bool incl0 = lq ? oincl : incl, incl1 = lq ? incl : oincl;
                prefix += lq ? osum : sum;
                if (!incl0) prefix += lq ? sum : osum;
                if (incl0 || incl1) break;
            }
        }
        if (last && lq == 0) st_status32(sst + (uint64_t)S * kRadix, kOsIncl | (prefix + own));
        if (lq == 0) s_off[ld] += prefix;
    }
    __syncthreads();
    // write each digit run with consecutive lanes (coalesced)
    const uint64_t tn = n > base ? min<uint64_t>(n - base, kPsTile) : 0;
#pragma unroll
    for (int j = 0; j < kRounds; ++j) {
        const uint32_t lp = j * kPsThreads + t;
        if (lp < tn) {
            const K k = skey[lp];
            const uint32_t dd = digit(k);
            const uint32_t pos = s_off[dd] + lp;
            // stays below n unless a look-back wait ran out (err is set);
            // then the write is dropped rather than sent out of bounds
            if (pos < n) {
                kout[pos] = k;
                if (HasVal) vout[pos] = sval[lp];
            }
        }
    }
}

// concurrent: other kernels may hold compute units while the passes run
// (work on another stream), so tiles take tickets in launch order
template <typename K, bool HasVal>
bool onesweep_passes(Ctx& c, K* k0, K* k1, uint32_t* v0, uint32_t* v1, const uint32_t* n_dev,
                     uint64_t n_max, int bits, uint32_t* state, uint32_t* err,
                     uint32_t spin_limit = kSpinLimit, bool concurrent = false);

// Look-back counts are 30-bit fields of the status words: a sort takes fewer
// than 2^30 keys.
constexpr uint64_t kOsMaxKeys = 1ull << 30;

// Sorts n keys (n on the device when n_dev != null, n_max bounds it) by bits
// [0, bits), stably, ping-ponging k0/k1 (v0/v1).  `state` must hold
// os_words(n_max, bits, HasVal) uint32 words, which the digit counting clears as far
// as the passes need it, with `clear_words` words at `clear` for the caller
// (a kernel for that alone took 2.1 us at 10^5 keys, 4.5 at 10^6);
// `concurrent` as for onesweep_passes.  Returns true if the result is in
// k1/v1.  Nothing runs for one key or no bits.
template <typename K, bool HasVal>
bool onesweep(Ctx& c, K* k0, K* k1, uint32_t* v0, uint32_t* v1, const uint32_t* n_dev,
              uint64_t n_max, int bits, uint32_t* state, uint32_t* err,
              uint32_t spin_limit = kSpinLimit, bool concurrent = false,
              uint32_t* clear = nullptr, uint32_t clear_words = 0) {
    if (n_max <= 1 || bits <= 0) return false;
    if (n_max >= kOsMaxKeys) fail(GV_EINVAL, "sort of 2^30 or more keys");
    const int passes = os_passes(bits);
    if (passes > 8) fail(GV_EINVAL, "too many radix passes");
    const uint64_t hg = os_hist_groups(n_max);
    const uint32_t hwords = (uint32_t)passes * kRadix;
    uint32_t* hist = state + os_zero_words(n_max, bits, HasVal);  // passes * 256 counters
    uint32_t* hpart = hist + hwords;      // per histogram workgroup
    c.launch("sort_hist", k_os_hist<K>, hg, kOsThreads, (const K*)k0, n_dev, n_max, passes, hpart,
             state, os_zero_words(n_max, bits, HasVal), clear, clear_words);
    c.launch("sort_hist", k_os_hist_sum, div_up(hwords, 16), kThreads, (const uint32_t*)hpart,
             (uint32_t)hg, hwords, hist, (const uint32_t*)nullptr, (unsigned long long*)nullptr,
             (const unsigned long long*)nullptr, (unsigned long long*)nullptr);
    return onesweep_passes<K, HasVal>(c, k0, k1, v0, v1, n_dev, n_max, bits, state, err,
                                      spin_limit, concurrent);
}

// Per-group digit counts of a sort whose histogram kernel is fused into the
// kernel that writes the keys: group g writes os_passes(bits) * kRadix counts
// at os_hpart(...) + g * os_passes(bits) * kRadix, for os_hist_groups(n_max)
// groups of kHistTile-key tiles (tile t to group t % groups).
inline uint32_t* os_hpart(uint32_t* state, uint64_t n_max, int bits) {
    return state + os_zero_words(n_max, bits) + (uint64_t)os_passes(bits) * kRadix;
}

// Adds the per-group counts into the pass histograms; with vpart, also adds
// os_hist_groups(n_max) per-group counts into *vtotal and the groups' 64-bit
// kpart sums into *ktotal.  One launch, also when there is nothing to sort.
inline void os_hist_sum(Ctx& c, uint32_t* state, uint64_t n_max, int bits, const uint32_t* vpart,
                        unsigned long long* vtotal, const unsigned long long* kpart,
                        unsigned long long* ktotal) {
    const uint32_t hwords = bits > 0 ? (uint32_t)os_passes(bits) * kRadix : 0u;
    c.launch("sort_hist", k_os_hist_sum, std::max<uint64_t>(div_up(hwords, 16), 1), kThreads,
             (const uint32_t*)os_hpart(state, n_max, bits), (uint32_t)os_hist_groups(n_max), hwords,
             state + os_zero_words(n_max, bits), vpart, vtotal, kpart, ktotal);
}

// The passes of onesweep, once the pass histograms are in the state.
template <typename K, bool HasVal>
bool onesweep_passes(Ctx& c, K* k0, K* k1, uint32_t* v0, uint32_t* v1, const uint32_t* n_dev,
                     uint64_t n_max, int bits, uint32_t* state, uint32_t* err,
                     uint32_t spin_limit, bool concurrent) {
    if (n_max <= 1 || bits <= 0) return false;
    if (n_max >= kOsMaxKeys) fail(GV_EINVAL, "sort of 2^30 or more keys");
    const int passes = os_passes(bits);
    if (passes > 8) fail(GV_EINVAL, "too many radix passes");
    const uint64_t nt = ps_tiles(n_max, HasVal), per = ps_status(n_max, HasVal) * kRadix;
    uint32_t* counters = state;           // 64 words
    uint32_t* hist = state + os_zero_words(n_max, bits, HasVal);  // passes * 256 counters
    auto kernel = k_os_pass<K, HasVal, kPsRounds>;
    const int rounds = ps_rounds(n_max, HasVal);
    if (rounds == kPsRoundsShort) kernel = k_os_pass<K, HasVal, kPsRoundsShort>;
    if constexpr (!HasVal) {
        if (rounds == kPsRoundsLong) kernel = k_os_pass<K, false, kPsRoundsLong>;
    }
    const int block_tiles = !concurrent && nt <= resident_grid(kernel, kPsThreads) ? 1 : 0;
    bool flip = false;
    for (int p = 0; p < passes; ++p) {
        K* kin = flip ? k1 : k0;
        K* kout = flip ? k0 : k1;
        uint32_t* vin = flip ? v1 : v0;
        uint32_t* vout = flip ? v0 : v1;
        c.launch("sort_pass", kernel, nt, kPsThreads, (const K*)kin, kout,
                 (const uint32_t*)vin, vout, n_dev, n_max, p * kRadixBits,
                 (const uint32_t*)(hist + (uint64_t)p * kRadix),
                 state + 64 + (uint64_t)p * per, counters + p, block_tiles, err, spin_limit);
        flip = !flip;
    }
    return flip;
}

static __global__ void k_zero_words(uint32_t* p, uint64_t n) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

inline void zero_words(Ctx& c, uint32_t* p, uint64_t n) {
    if (n) c.launch("zero", k_zero_words, std::min<uint64_t>(div_up(n, kThreads), 4096), kThreads, p, n);
}

// ---------------------------------------------------------------- rank sort
// Sort by rank of at most kRankMax keys in one kernel.  A workgroup owns
// kRankTile keys, a wave's worth, which it orders by counting (every wave
// holds them all and compares its share), and reads all the other keys: each
// is placed among the tile's by a search in LDS and counted there, and the
// running sum of the counts is how many foreign keys stand before each of the
// tile's.  Equal keys rank in input order, so the sort is stable.  Every
// workgroup makes the keys anew from the input, so packing is not a kernel of
// its own; a thread has the inputs of all its kRows keys in flight at once,
// ahead of the tile's ordering.
//
// Work grows with n^2 / kRankTile searches, but over the whole chip and
// without a chain of passes.  Bound: the searches past some thousand keys, the
// latency input -> activity word below: 1000 pairs 9.8 -> 4.9 us, 10^4 pairs
// 18.5 -> 13.6 (3.2 of them the keys) against tiles of 256 keys that read the
// others in turn; packing, digit sums and five radix passes took 56.  Comparing
// the upper 32 bits first (10.6 us) and eight copies of the counts (10.1) were
// no better.
//
// P: Raw raw(i) input i; uint64_t key(raw) its key (below 2^63); void own(i,
// key) once per input; void begin(t, nt) by the first workgroup; bool
// counted(key) and void totals(n, sum): the number and the mix64 sum of the
// counted keys, by one thread.
constexpr uint32_t kRankTile = 64;
constexpr uint64_t kRankMax = 16384;
constexpr uint32_t kRankThreads = 1024;
constexpr uint32_t kRankRows = kRankMax / kRankThreads;

template <typename P, uint32_t kRows>
__global__ __launch_bounds__(kRankThreads) void k_rank_sort(P pk, uint32_t n, uint64_t* keys,
                                                            uint32_t* vals) {
    constexpr uint32_t W = kRankThreads / 64;
    static_assert(kRankTile == 64 && kRankTile % W == 0, "a tile key per lane");
    __shared__ uint64_t s_srt[kRankTile];
    __shared__ uint32_t s_q[W][kRankTile], s_idx[kRankTile], s_add[kRankTile];
    __shared__ unsigned long long s_tot[2];
    const uint32_t t = threadIdx.x, lane = lane_id();
    const uint32_t w = __builtin_amdgcn_readfirstlane(t >> 6);
    const uint32_t tb = blockIdx.x * kRankTile;
    const bool first = blockIdx.x == 0;
    // unconditional loads at clamped positions
    const typename P::Raw mine = pk.raw(min(tb + lane, n - 1));
    typename P::Raw raw[kRows];
#pragma unroll
    for (uint32_t u = 0; u < kRows; ++u) raw[u] = pk.raw(min(u * kRankThreads + t, n - 1));
    if (first) {
        pk.begin(t, kRankThreads);
        if (t < 2) s_tot[t] = 0ull;
    }
    uint64_t my = pk.key(mine);
    uint64_t x[kRows];
#pragma unroll
    for (uint32_t u = 0; u < kRows; ++u) x[u] = pk.key(raw[u]);
    if (tb + lane >= n) my = ~0ull;  // past every key
    {
        uint32_t c = 0;
#pragma unroll
        for (uint32_t i = 0; i < kRankTile / W; ++i) {
            const uint32_t m = w * (kRankTile / W) + i;
            const uint64_t o = (uint64_t)__builtin_amdgcn_readlane((uint32_t)(my >> 32), m) << 32 |
                               (uint32_t)__builtin_amdgcn_readlane((uint32_t)my, m);
            c += (o < my) | ((o == my) & (m < lane));
        }
        s_q[w][lane] = c;
    }
    if (t < kRankTile) s_add[t] = 0;
    __syncthreads();
    if (w == 0) {
        uint32_t r = 0;
#pragma unroll
        for (uint32_t i = 0; i < W; ++i) r += s_q[i][lane];
        s_srt[r] = my;
        s_idx[r] = lane;
        if (tb + lane < n) pk.own(tb + lane, my);
    }
    __syncthreads();
    unsigned long long cnt = 0, sum = 0;
    if (first) {
#pragma unroll
        for (uint32_t u = 0; u < kRows; ++u)
            if (u * kRankThreads + t < n && pk.counted(x[u])) {
                ++cnt;
                sum += mix64(x[u]);
            }
    }
    constexpr uint32_t kU = kRows < 4 ? kRows : 4;  // searches in lockstep
#pragma unroll
    for (uint32_t u0 = 0; u0 < kRows; u0 += kU) {
        if (u0 * kRankThreads >= n) break;
        uint32_t p[kU];  // byte offset into s_srt
#pragma unroll
        for (uint32_t u = 0; u < kU; ++u) {
            // an equal key of the tile stands before a later foreign key
            x[u0 + u] += (u0 + u) * kRankThreads + t < tb ? 0ull : 1ull;
            p[u] = 0;
        }
        auto at = [&](uint32_t o) { return *(const uint64_t*)((const char*)s_srt + o); };
#pragma unroll
        for (uint32_t half = 8 * kRankTile / 2; half >= 8; half >>= 1) {
#pragma unroll
            for (uint32_t u = 0; u < kU; ++u)
                p[u] += at(p[u] + half - 8) < x[u0 + u] ? half : 0u;
        }
#pragma unroll
        for (uint32_t u = 0; u < kU; ++u) {
            const uint32_t j = (u0 + u) * kRankThreads + t;
            p[u] += at(p[u]) < x[u0 + u] ? 8u : 0u;
            if (j < n && j / kRankTile != blockIdx.x && p[u] < 8 * kRankTile)
                atomicAdd(&s_add[p[u] / 8], 1u);
        }
    }
    __syncthreads();
    if (w == 0) {
        const uint32_t at = lane + wave_incl_scan(s_add[lane]);
        const uint32_t i = tb + s_idx[lane];
        if (i < n) {
            keys[at] = s_srt[lane];
            if (vals) vals[at] = i;
        }
    }
    if (first) {
        cnt = wave_sum(cnt);
        sum = wave_sum(sum);
        if (lane == 0) {
            atomicAdd(&s_tot[0], cnt);
            atomicAdd(&s_tot[1], sum);
        }
        __syncthreads();
        if (t == 0) pk.totals(s_tot[0], s_tot[1]);
    }
}

// the keys of pk, made once (k) for a kernel whose workgroups all read them
template <typename P>
struct RankPacked {
    using Raw = uint64_t;
    P pk;
    const uint64_t* k;
    __device__ Raw raw(uint64_t i) const { return k[i]; }
    __device__ uint64_t key(Raw r) const { return r; }
    __device__ void own(uint64_t i, uint64_t key) const { pk.own(i, key); }
    __device__ void begin(uint32_t t, uint32_t nt) const { pk.begin(t, nt); }
    __device__ bool counted(uint64_t key) const { return pk.counted(key); }
    __device__ void totals(unsigned long long n, unsigned long long sum) const {
        pk.totals(n, sum);
    }
};

template <typename P>
__global__ __launch_bounds__(kThreads) void k_rank_pack(P pk, uint32_t n, uint64_t* packed) {
    const uint32_t i = blockIdx.x * kThreads + threadIdx.x;
    if (i < n) packed[i] = pk.key(pk.raw(i));
}

// calls f with the kernel for n keys, at most kMost rows of them
template <typename P, uint32_t kMost, uint32_t kRows = 1, typename F>
void with_rank_sort(uint64_t n, F&& f) {
    if constexpr (kRows < kMost) {
        if (n > kRows * kRankThreads) return with_rank_sort<P, kMost, 2 * kRows>(n, f);
    }
    f(k_rank_sort<P, kRows>);
}

// the n > 0 keys of pk in order, and (vals not null) their input positions;
// packed: n words of scratch.  Keys that take gathered reads (P::kGathers: the activity
// words, a line per lane) are made by a kernel of their own past
// kRankFused keys: made anew by every workgroup they cost 12 of 18 us at 10^4
// pairs, below that limit less than the launch.
constexpr uint64_t kRankFused = 4 * kRankThreads;
template <typename P>
void rank_sort(Ctx& c, const char* name, P pk, uint64_t n, uint64_t* packed, uint64_t* keys,
               uint32_t* vals) {
    if (n > kRankMax) fail(GV_EINVAL, "too many keys to sort by rank");
    const uint64_t nt = div_up(n, kRankTile);
    if constexpr (P::kGathers) {
        if (n > kRankFused) {
            c.launch(name, k_rank_pack<P>, div_up(n, kThreads), kThreads, pk, (uint32_t)n, packed);
            auto run = [&](auto kernel) {
                c.launch(name, kernel, nt, kRankThreads, RankPacked<P>{pk, packed}, (uint32_t)n,
                         keys, vals);
            };
            return with_rank_sort<RankPacked<P>, kRankRows, 8>(n, run);
        }
    }
    with_rank_sort<P, P::kGathers ? kRankFused / kRankThreads : kRankRows>(n, [&](auto kernel) {
        c.launch(name, kernel, nt, kRankThreads, pk, (uint32_t)n, keys, vals);
    });
}

}  // namespace gv
