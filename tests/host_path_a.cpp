// Failure events against a device that this program plays: which way the search's ids come, after errors of every kind, and what a call leaves
// behind.  Built with csrc/path_a.cpp and csrc/arc.cpp by test_path_a_host.py.  Prints "ok" or the first violated expectation.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "evospec.h"
#include "evospec_arc.h"
#include "launch.hpp"

#define REQUIRE(cond) do { if (!(cond)) { std::printf("FAILED line %d: %s\n", __LINE__, #cond); return 1; } } while (0)

namespace {
enum Search { kWorks, kLaunchFails, kIdsMissing } g_search = kWorks;
bool g_sync_fails = false, g_recording = false, g_alone = false;
int g_copies = 0, g_blocks = 0, g_refused = 0;
}  // namespace

// ---- the device
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
    if (!g_alone) ++g_refused;                                    // (as another thread's recording would have it)
    *p = std::calloc(1, n);
    ++g_blocks;
    return hipSuccess;
}
hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return g_sync_fails || g_recording ? hipErrorUnknown : hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
    *s = g_recording ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* mode) {
    const hipStreamCaptureMode was = g_alone ? hipStreamCaptureModeRelaxed : hipStreamCaptureModeGlobal;
    g_alone = *mode == hipStreamCaptureModeRelaxed;
    *mode = was;
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind, hipStream_t) {
    std::memcpy(dst, src, n);
    ++g_copies;
    return hipSuccess;
}
hipError_t hipMemcpyWithStream(void* dst, const void* src, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(dst, src, n); return hipSuccess; }

// ---- the library beside it
extern "C" int evospec_workspace_bytes(int, int, int, int, size_t* out) { *out = 256; return EVOSPEC_OK; }
extern "C" int evospec_active_lmhead_topk(const void*, int, int, const void*, const int32_t*, int, int, int k, float* vals, int32_t* ids, float* logz,
                                          void*, size_t, void*) {
    if (g_search == kLaunchFails) return EVOSPEC_HIP_ERROR;
    for (int i = 0; i < k; ++i) {
        vals[i] = -(float)i;
        if (g_search == kWorks || i > 0) ids[i] = 7 * i;
    }
    *logz = 1.f;
    return EVOSPEC_OK;
}
extern "C" int evospec_active_gather(const void*, int, int, const int32_t*, const int32_t*, int, void*, int32_t*, int, int, void*) { return EVOSPEC_OK; }
namespace evospec {
hipError_t launch_gather_inline(const void*, int, int, const int32_t*, const int32_t*, int, void*, int32_t*, int, hipStream_t, bool) { return hipSuccess; }
int record_hip_error(hipError_t) { return EVOSPEC_HIP_ERROR; }
}  // namespace evospec

int main() {
    constexpr int V = 1000, d = 64, n_core = 100, cap = 64, k = 10;
    std::vector<int32_t> core(n_core), act(n_core + cap), top{900, 901};
    for (int i = 0; i < n_core; ++i) core[i] = 500 + i;
    std::vector<int64_t> row_ptr(V + 1, 0);
    std::vector<int32_t> col(1, 0);
    alignas(16) static unsigned char mem[1 << 16];
    evospec_arc_config cfg;
    evospec_arc_default_config(&cfg);
    cfg.capacity = cap; cfg.p0 = cap / 2; cfg.ghost_capacity = cap; cfg.max_insert = 16; cfg.slot_base = n_core;
    evospec_arc* arc = nullptr;
    REQUIRE(evospec_arc_create(&cfg, core.data(), n_core, &arc) == EVOSPEC_OK);
    auto event = [&]() {
        int32_t slots[16], ids[16];
        int n = 0;
        return evospec_path_a_event(arc, mem, d, mem, V, top.data(), (int)top.size(), k, row_ptr.data(), col.data(), 4, mem, act.data(), n_core + cap,
                                    EVOSPEC_ROW_MAJOR, mem, sizeof mem, nullptr, slots, ids, &n);
    };
    REQUIRE(event() == EVOSPEC_OK && g_copies == 0 && g_blocks == 1 && g_refused == 0 && !g_alone);
    // errors that leave nothing under way cost no place, however many there are
    for (int i = 0; i < 40; ++i) {
        g_search = i % 2 ? kLaunchFails : kIdsMissing;
        REQUIRE(event() == EVOSPEC_HIP_ERROR);
    }
    g_search = kWorks;
    REQUIRE(event() == EVOSPEC_OK && g_copies == 0);
    // a stream that records a graph is refused, by way of the copy
    g_recording = true;
    for (int i = 0; i < 40; ++i) REQUIRE(event() == EVOSPEC_HIP_ERROR);
    g_recording = false;
    g_copies = 0;
    REQUIRE(event() == EVOSPEC_OK && g_copies == 0);
    // one whose work may still be under way keeps its place for good; past the last place ids are copied
    g_search = kIdsMissing;
    g_sync_fails = true;
    for (int i = 0; i < 16; ++i) REQUIRE(event() == EVOSPEC_HIP_ERROR && g_copies == 0);
    g_search = kWorks;
    g_sync_fails = false;
    REQUIRE(event() == EVOSPEC_OK && g_copies == 1 && g_blocks == 1);
    evospec_arc_destroy(arc);
    std::printf("ok\n");
    return 0;
}
