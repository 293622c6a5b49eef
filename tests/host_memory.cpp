// The library's device allocations against a card simulated on the host: the
// HIP calls that they make are defined here.  Each check prints its name and
// "ok", or what it found.
#include <cstdlib>
#include <cstring>
#include <map>

#include "gv_host.h"

static size_t g_card = (size_t)1 << 40, g_used = 0, g_allocs = 0;
static std::map<void*, size_t> g_bufs;
static hipError_t g_last = hipSuccess;

extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
    if (g_used + n > g_card) return g_last = hipErrorOutOfMemory;
    *p = std::malloc(1);
    g_bufs[*p] = n;
    g_used += n;
    ++g_allocs;
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    auto it = g_bufs.find(p);
    if (it == g_bufs.end()) return g_last = hipErrorInvalidValue;
    g_used -= it->second;
    g_bufs.erase(it);
    std::free(p);
    return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError() {
    const hipError_t e = g_last;
    g_last = hipSuccess;
    return e;
}
const char* hipGetErrorString(hipError_t) { return "simulated"; }
}

using namespace gv;
constexpr size_t MiB = (size_t)1 << 20;

static int code_of(const std::function<void()>& f) {
    try {
        f();
    } catch (const Error& e) {
        return e.code;
    }
    return GV_OK;
}

// a buffer that could not grow is gone, and whoever recorded it can tell
static const char* scratch_growth_fails() {
    Scratch s;
    s.ensure(8 * MiB, nullptr);
    const uint64_t gen = s.gen;
    g_card = g_used + 4 * MiB;
    if (code_of([&] { s.ensure(64 * MiB, nullptr); }) != GV_ENOMEM) return "no error";
    if (s.ptr || s.cap) return "a pointer to a released buffer";
    if (s.gen == gen) return "the old buffer's generation";
    g_card = (size_t)1 << 40;
    const uint64_t failed = s.gen;
    s.ensure(8 * MiB, nullptr);
    if (!s.ptr || s.gen == failed || s.gen == gen) return "a generation seen before";
    s.release(true);
    return nullptr;
}

// any request of the library is served while buffers are only kept
static const char* requests_empty_the_cache() {
    for (size_t want : {48 * MiB, 8 * MiB, 65 * MiB}) {
        void *a = nullptr, *b = nullptr;
        dev_malloc(&a, 64 * MiB, "kept");
        dev_free(a, true);
        if (g_used != 64 * MiB) return "not kept";
        g_card = 66 * MiB;
        if (code_of([&] { dev_malloc(&b, want, "request"); }) != GV_OK) return "a request failed";
        dev_free(b, false);
        dev_malloc(&a, 64 * MiB, "kept");
        dev_free(a, true);
        if (dev_alloc(&b, want) != hipSuccess) return "a plain request failed";
        hipFree(b);
        if (g_used) return "still held";
        // one that does not fit at all leaves no error to be found later
        if (code_of([&] { dev_malloc(&b, 4 * want + 70 * MiB, "too much"); }) != GV_ENOMEM)
            return "no error";
        if (hipGetLastError() != hipSuccess) return "an error left behind";
        g_card = (size_t)1 << 40;
    }
    return nullptr;
}

// what is kept is bounded, is found again by size, and ends by age or request
static const char* bounded_and_given_back() {
    std::vector<void*> p(12);
    for (void*& x : p) dev_malloc(&x, 512 * MiB, "pool");
    for (void* x : p) dev_free(x, true);
    if (g_used > kCacheMax) return "more than the bound";
    if (!g_used) return "nothing kept";
    void* x = nullptr;
    dev_malloc(&x, 420 * MiB, "fits one of them");
    if (std::find(p.begin(), p.end(), x) == p.end()) return "a new buffer";
    size_t held = g_used;
    dev_free(x, false);  // (its streams were not waited for)
    if (g_used != held - 512 * MiB) return "kept though it may be in use";
    held = g_used;
    if (dev_release_cached() != held || g_used) return "not given back";
    dev_malloc(&x, 64 * MiB, "old");
    dev_free(x, true);
    for (uint64_t i = 0; i <= kCacheAge; ++i) {
        void* y = nullptr;
        dev_malloc(&y, 200 * MiB, "passing by");
        dev_free(y, false);
    }
    if (g_used) return "kept for ever";
    dev_malloc(&x, kCacheMax + 64 * MiB, "past the bound");
    dev_free(x, true);
    return g_used ? "kept past the bound" : nullptr;
}

// a scratch buffer of a few MiB that grows and goes, graph after graph, comes
// from what is kept
static const char* growing_scratch_is_kept() {
    size_t first = 0;
    for (int i = 0; i < 8; ++i) {
        Scratch s;
        s.ensure(2 * MiB, nullptr);
        s.ensure(4 * MiB, nullptr);
        s.release(true);
        if (i == 0) first = g_allocs;
    }
    if (g_allocs != first) return "allocated again";
    dev_release_cached();
    return g_used ? "still held" : nullptr;
}

// an error is reported by the call that met it, and by no other
static const char* error_stays_with_its_call() {
    for (hipError_t e : {hipErrorInvalidValue, hipErrorOutOfMemory}) {
        g_last = e;  // as the runtime keeps it
        const int want = e == hipErrorOutOfMemory ? GV_ENOMEM : GV_EDEVICE;
        if (code_of([&] { hip_check(e, "a call"); }) != want) return "another code";
        if (hipGetLastError() != hipSuccess) return "left for the next call";
    }
    return nullptr;
}

int main(int argc, char** argv) {
    struct {
        const char* name;
        const char* (*run)();
    } checks[] = {{"scratch_growth_fails", scratch_growth_fails},
                  {"requests_empty_the_cache", requests_empty_the_cache},
                  {"bounded_and_given_back", bounded_and_given_back},
                  {"growing_scratch_is_kept", growing_scratch_is_kept},
                  {"error_stays_with_its_call", error_stays_with_its_call}};
    for (auto& c : checks)
        if (argc > 1 && !std::strcmp(argv[1], c.name)) {
            const char* bad = c.run();
            std::printf("%s: %s\n", c.name, bad ? bad : "ok");
            return bad ? 1 : 0;
        }
    return 2;
}
