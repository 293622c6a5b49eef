// gv_host.h -- host-side launch context, error handling and scratch carving.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cstdio>
#include <cstring>
#include <functional>
#include <mutex>
#include <string>
#include <utility>
#include <vector>

#include "../../include/graphvine.h"

namespace gv {

// Internal failures carry a GV_* code; they are caught at the C ABI.
struct Error {
    int code;
    const char* what;
};

[[noreturn]] inline void fail(int code, const char* what) { throw Error{code, what}; }

// Text of the last internal failure on this thread ("call: HIP error").
inline char* last_error_text() {
    static thread_local char buf[256] = "";
    return buf;
}

inline void hip_check(hipError_t e, const char* what) {
    if (e == hipSuccess) return;
    // the runtime keeps the error until it is asked for: left there, the next
    // launch's check would report it for another graph
    (void)hipGetLastError();
    std::snprintf(last_error_text(), 256, "%s: %s", what, hipGetErrorString(e));
    if (e == hipErrorOutOfMemory || e == hipErrorMemoryAllocation) fail(GV_ENOMEM, what);
    fail(GV_EDEVICE, what);
}

// Workgroups of `kernel` (launched with `block` threads) that the current
// device holds at once: compute units times resident workgroups per unit.
// Kernels that loop over their work size their grid with it, so that no
// workgroup waits for a second round.  Cached per kernel and device.
template <typename... KArgs>
uint64_t resident_grid(void (*kernel)(KArgs...), uint32_t block) {
    struct Entry {
        const void* k;
        int dev;
        uint32_t block;
        uint64_t grid;
    };
    static std::mutex mu;
    static std::vector<Entry> cache;
    int dev = 0;
    hip_check(hipGetDevice(&dev), "hipGetDevice");
    std::lock_guard<std::mutex> lock(mu);
    for (const Entry& e : cache)
        if (e.k == (const void*)kernel && e.dev == dev && e.block == block) return e.grid;
    int cus = 0, per = 0;
    hip_check(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev),
              "hipDeviceGetAttribute");
    hip_check(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kernel, (int)block, 0),
              "hipOccupancyMaxActiveBlocksPerMultiprocessor");
    const uint64_t grid = (uint64_t)std::max(cus, 1) * (uint64_t)std::max(per, 1);
    cache.push_back({(const void*)kernel, dev, block, grid});
    return grid;
}

// Kernel launches go through Ctx so that they can be timed with HIP events on
// the graph's stream when profiling is enabled.  With every kernel timed, each
// launch gets its own pair of events.  When only one kernel name is timed,
// one pair of events brackets each run of consecutive launches of it (the
// radix passes of a sort are one run): an event record costs GPU time of its
// own, and a run shares one, so the average per launch stays close to the
// kernels' own durations.
struct Ctx {
    hipStream_t stream = nullptr;
    uint64_t seq = 0;  // operations queued so far (launches, recorded graphs)
    // device state of the one-kernel small scans (a ChainState) and the word
    // their bounded waits flag when one runs out; null: two-kernel scans only
    void* chain = nullptr;
    uint32_t* chain_err = nullptr;
    bool prof = false;
    std::string only;  // when non-empty, only launches of this name are timed
    struct Rec {
        const char* name;
        hipEvent_t e0, e1;
        uint64_t launches;
    };
    hipEvent_t run_e0 = nullptr;   // open run of the timed kernel
    const char* run_name = nullptr;
    uint64_t run_n = 0;
    std::vector<Rec> recs;
    std::vector<hipEvent_t> spare;
    struct Sum {
        std::string name;
        uint64_t launches;
        double ms;
    };
    std::vector<Sum> sums;

    hipEvent_t event() {
        if (!spare.empty()) {
            hipEvent_t e = spare.back();
            spare.pop_back();
            return e;
        }
        hipEvent_t e;
        hip_check(hipEventCreate(&e), "hipEventCreate");
        return e;
    }

    // Closes an open run of the timed kernel (records its end event).
    void close_run() {
        if (!run_e0) return;
        hipEvent_t e1 = event();
        hip_check(hipEventRecord(e1, stream), "hipEventRecord");
        recs.push_back({run_name, run_e0, e1, run_n});
        run_e0 = nullptr;
        run_n = 0;
    }

    // Fold finished records into per-name sums (synchronises the stream).
    void collect() {
        close_run();
        if (recs.empty()) return;
        hip_check(hipStreamSynchronize(stream), "hipStreamSynchronize");
        for (auto& r : recs) {
            float ms = 0.f;
            hip_check(hipEventElapsedTime(&ms, r.e0, r.e1), "hipEventElapsedTime");
            bool found = false;
            for (auto& s : sums)
                if (s.name == r.name) {
                    s.launches += r.launches;
                    s.ms += ms;
                    found = true;
                    break;
                }
            if (!found) sums.push_back({r.name, r.launches, (double)ms});
            spare.push_back(r.e0);
            spare.push_back(r.e1);
        }
        recs.clear();
    }

    void release() {
        if (run_e0) hipEventDestroy(run_e0);
        run_e0 = nullptr;
        for (auto& r : recs) {
            hipEventDestroy(r.e0);
            hipEventDestroy(r.e1);
        }
        recs.clear();
        for (auto e : spare) hipEventDestroy(e);
        spare.clear();
    }

    template <typename... KArgs, typename... Args>
    void launch(const char* name, void (*kernel)(KArgs...), uint64_t grid, uint32_t block,
                Args... args) {
        if (grid == 0) return;
        if (grid > 0x7fffffffull) fail(GV_EINVAL, "grid too large");
        ++seq;
        const bool timed = prof && (only.empty() || only == name);
        if (prof && !only.empty()) {
            // runs of the one timed kernel
            if (!timed) {
                close_run();
            } else if (!run_e0) {
                run_e0 = event();
                run_name = name;
                hip_check(hipEventRecord(run_e0, stream), "hipEventRecord");
            }
            hipLaunchKernelGGL(kernel, dim3((uint32_t)grid), dim3(block), 0, stream, args...);
            hip_check(hipGetLastError(), name);
            if (timed) ++run_n;
            if (recs.size() > 4096) collect();
            return;
        }
        hipEvent_t e0 = nullptr;
        if (timed) {
            e0 = event();
            hip_check(hipEventRecord(e0, stream), "hipEventRecord");
        }
        hipLaunchKernelGGL(kernel, dim3((uint32_t)grid), dim3(block), 0, stream, args...);
        hip_check(hipGetLastError(), name);
        if (timed) {
            hipEvent_t e1 = event();
            hip_check(hipEventRecord(e1, stream), "hipEventRecord");
            recs.push_back({name, e0, e1, 1});
            if (recs.size() > 4096) collect();
        }
    }
};

// Carves typed arrays out of one device buffer.  With base == nullptr it only
// measures, so a caller can size the buffer first and carve second.
struct Carver {
    char* base;
    size_t used = 0;
    explicit Carver(void* b) : base((char*)b) {}
    template <typename T>
    T* take(uint64_t n) {
        used = (used + 255) & ~size_t(255);
        T* p = base ? (T*)(base + used) : nullptr;
        used += (size_t)n * sizeof(T);
        return p;
    }
};

// Device buffers from 2 MiB on (a graph's pool and scratch) go through a cache:
// a freed one is kept and given to the next request it fits (at most a
// quarter larger).  hipFree of a buffer past 64 MiB takes about 230 us here,
// hipMalloc 40 us, and the driver hands freed memory back slowly: a program
// that builds and drops graphs of 1 GB each waited 18 ms per graph once the
// card's 288 GB had been through its hands.  What is kept is bounded
// (kCacheMax over all devices, the oldest goes first), is freed when any
// allocation of the library does not fit the card or the program asks for it
// (gv_release_cached), and is dropped when it was passed over by kCacheAge
// requests and frees.  Callers free a buffer only after waiting for the streams
// that used it, so the next owner may use any stream.  From 2 MiB on each
// allocation and free goes to the driver: a graph with a pool of 100 MiB made,
// given 1000 pairs (its scratch grows from 2.5 to 4 MB) and destroyed takes 208
// us, 764 with only the buffers past 32 MiB kept (700 before any were).
constexpr size_t kCacheMin = (size_t)2 << 20;
constexpr size_t kCacheMax = (size_t)4 << 30;
constexpr uint64_t kCacheAge = 64;
struct DevCache {
    struct Buf {
        void* p;
        size_t bytes;
        int dev;
        uint64_t stamp;
    };
    std::mutex mu;
    std::vector<Buf> idle, live;
    uint64_t clock = 0;

    // takes out of the idle list what is too old or past the bound (the lock
    // is held; the caller frees it afterwards)
    void trim(std::vector<Buf>& out, size_t bound) {
        size_t total = 0;
        for (size_t i = idle.size(); i-- > 0;) {  // newest last
            total += idle[i].bytes;
            if (total > bound || clock - idle[i].stamp > kCacheAge) {
                total -= idle[i].bytes;
                out.push_back(idle[i]);
                idle.erase(idle.begin() + (long)i);
            }
        }
    }
};

inline DevCache& dev_cache() {
    static DevCache* c = new DevCache;  // outlives every graph
    return *c;
}

inline void dev_free_all(const std::vector<DevCache::Buf>& bufs) {
    for (const DevCache::Buf& b : bufs) (void)hipFree(b.p);
}

// Frees everything kept; returns how many bytes that was.
inline size_t dev_release_cached() {
    DevCache& c = dev_cache();
    std::vector<DevCache::Buf> old;
    {
        std::lock_guard<std::mutex> lock(c.mu);
        old.reserve(c.idle.size());
        c.trim(old, 0);
    }
    dev_free_all(old);
    size_t total = 0;
    for (const DevCache::Buf& b : old) total += b.bytes;
    return total;
}

// Every device allocation of the library: what is kept goes back to the card
// before a request fails.  (A failure leaves no error behind for the check of
// the next launch to find.)
inline hipError_t dev_alloc(void** out, size_t bytes) {
    hipError_t e = hipMalloc(out, bytes);
    if (e == hipSuccess) return e;
    (void)hipGetLastError();
    if (!dev_release_cached()) return e;
    e = hipMalloc(out, bytes);
    if (e != hipSuccess) (void)hipGetLastError();
    return e;
}

// a buffer from the cache where it has one, for dev_free to take back
inline void dev_malloc(void** out, size_t bytes, const char* what) {
    if (bytes < kCacheMin) {
        hip_check(dev_alloc(out, bytes), what);
        return;
    }
    int dev = 0;
    hip_check(hipGetDevice(&dev), "hipGetDevice");
    DevCache& c = dev_cache();
    std::vector<DevCache::Buf> old;
    bool got = false;
    {
        std::lock_guard<std::mutex> lock(c.mu);
        ++c.clock;
        size_t best = c.idle.size();
        for (size_t i = 0; i < c.idle.size(); ++i) {
            const DevCache::Buf& b = c.idle[i];
            if (b.dev == dev && b.bytes >= bytes && b.bytes <= bytes + bytes / 4 &&
                (best == c.idle.size() || b.bytes < c.idle[best].bytes))
                best = i;
        }
        c.live.reserve(c.live.size() + 1);
        if (best < c.idle.size()) {
            *out = c.idle[best].p;
            c.live.push_back(c.idle[best]);
            c.idle.erase(c.idle.begin() + (long)best);
            got = true;
        }
        old.reserve(c.idle.size());
        c.trim(old, kCacheMax);
    }
    dev_free_all(old);
    if (got) return;
    hip_check(dev_alloc(out, bytes), what);
    std::lock_guard<std::mutex> lock(c.mu);
    try {
        c.live.push_back({*out, bytes, dev, 0});
    } catch (...) {
        // not listed: dev_free then frees it at once
    }
}

// `reuse`: the streams that used the buffer were waited for
inline void dev_free(void* p, bool reuse) {
    if (!p) return;
    DevCache& c = dev_cache();
    std::vector<DevCache::Buf> old;
    {
        std::lock_guard<std::mutex> lock(c.mu);
        ++c.clock;
        for (size_t i = 0; i < c.live.size(); ++i) {
            if (c.live[i].p != p) continue;
            DevCache::Buf b = c.live[i];
            c.live.erase(c.live.begin() + (long)i);
            if (reuse && b.bytes <= kCacheMax) {
                b.stamp = c.clock;
                try {
                    old.reserve(c.idle.size() + 1);
                    c.idle.push_back(b);
                    p = nullptr;
                } catch (...) {
                }
            }
            break;
        }
        if (!p) c.trim(old, kCacheMax);
    }
    dev_free_all(old);
    if (p) (void)hipFree(p);
}

// Growable device scratch buffer owned by a graph.
struct Scratch {
    void* ptr = nullptr;
    size_t cap = 0;
    uint64_t gen = 0;  // counts the buffers had and given up
    void ensure(size_t bytes, hipStream_t s) {
        if (bytes <= cap) return;
        if (ptr) {
            hip_check(hipStreamSynchronize(s), "hipStreamSynchronize");
            // (also when the allocation below fails: a plan recorded on the
            // old buffer, which may be another graph's by then, is refused)
            ++gen;
            dev_free(ptr, true);
            ptr = nullptr;
            cap = 0;
        }
        size_t want = bytes + bytes / 4 + (1 << 20);
        dev_malloc(&ptr, want, "hipMalloc scratch");
        cap = want;
        ++gen;
    }
    void release(bool reuse) {
        dev_free(ptr, reuse);
        ptr = nullptr;
        cap = 0;
    }
};

inline uint64_t div_up(uint64_t a, uint64_t b) { return (a + b - 1) / b; }

}  // namespace gv
