// The library's device allocations against a card simulated on the host: the
// HIP calls that they make are defined here.  Each check prints its name and
// "ok", or what it found.
#include <cstdlib>
#include <cstring>
#include <map>

#include "gv_host.h"

static size_t g_card = (size_t)1 << 40, g_used = 0;
static std::map<void*, size_t> g_bufs;
static hipError_t g_last = hipSuccess;

extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
    if (g_used + n > g_card) return g_last = hipErrorOutOfMemory;
    *p = std::malloc(1);
    g_bufs[*p] = n;
    g_used += n;
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

int main(int argc, char** argv) {
    struct {
        const char* name;
        const char* (*run)();
    } checks[] = {{"scratch_growth_fails", scratch_growth_fails}};
    for (auto& c : checks)
        if (argc > 1 && !std::strcmp(argv[1], c.name)) {
            const char* bad = c.run();
            std::printf("%s: %s\n", c.name, bad ? bad : "ok");
            return bad ? 1 : 0;
        }
    return 2;
}
