// A HIP runtime and kernel launchers of a device that computes nothing, for
// tests of the library's host code (tess_api.cpp) without a GPU: device memory
// is a budget in bytes, a failed allocation leaves the runtime's last error
// set until it is read, every launcher returns that error, and calls that a
// stream capture does not allow fail.  What the host code asked for (forms,
// tiles, capacities, graphs) is recorded for the tests.  Test code only.
#include "tess_internal.h"

#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

namespace {
struct Block {
    size_t bytes;
    bool real;  // small blocks are backed by host memory (read back by the host code)
};
std::map<char *, Block> g_blocks;
size_t g_held = 0, g_budget = ~(size_t)0;
char *g_next = reinterpret_cast<char *>((uintptr_t)1 << 44);
hipError_t g_last = hipSuccess;
bool g_user_capture = false;  // the caller's stream is being captured
int g_own_capture = 0;
unsigned long long g_pairs_per_tile = 1, g_own_count = 0;

hipError_t result(hipError_t e) {
    if (e != hipSuccess) g_last = e;
    return e;
}
hipError_t launched() {
    const hipError_t e = g_last;
    g_last = hipSuccess;
    return e;
}
constexpr size_t kReal = (size_t)1 << 20;
}  // namespace

// what the last calls asked for
extern "C" {
struct FakeLog {
    long long setups, edge_setups, stack_setups, rasters, direct_rasters, counting_rasters;
    long long mallocs, frees, failed_mallocs, graphs, graph_launches, illegal;
    int32_t edges, Th, Tw, chunk, block, nstack;  // of the last image
    int64_t ntet, stored;
    double crease_bmax, bmax_per_q;
    unsigned long long cap, max_items;
    int64_t own_room;  // payloads for own records of the last image by edges
};
FakeLog fake_log;
void fake_reset() { std::memset(&fake_log, 0, sizeof(fake_log)); }
size_t fake_held() { return g_held; }
void fake_budget(size_t bytes) { g_budget = bytes; }
void fake_capturing(int on) { g_user_capture = on != 0; }
// pairs of every list and own records the next images report
void fake_counts(unsigned long long pairs_per_list, unsigned long long own) {
    g_pairs_per_tile = pairs_per_list;
    g_own_count = own;
}
int fake_last_error() { return (int)g_last; }
}

// ------------------------------------------------------------- runtime
extern "C" {
hipError_t hipGetLastError() { return launched(); }
const char *hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : e == hipSuccess ? "no error" : "error"; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) {
    if (g_user_capture) {
        ++fake_log.illegal;
        return result(hipErrorStreamCaptureUnsupported);
    }
    if (n > g_budget || g_held > g_budget - n) {
        ++fake_log.failed_mallocs;
        return result(hipErrorOutOfMemory);
    }
    ++fake_log.mallocs;
    const bool real = n <= kReal;
    char *q = real ? (char *)calloc(n ? n : 1, 1) : g_next;
    if (!real) g_next += (n + 4095) / 4096 * 4096;
    g_blocks[q] = Block{n, real};
    g_held += n;
    *p = q;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    if (!p) return hipSuccess;
    if (g_user_capture) {
        ++fake_log.illegal;
        return result(hipErrorStreamCaptureUnsupported);
    }
    auto it = g_blocks.find((char *)p);
    if (it == g_blocks.end()) return result(hipErrorInvalidValue);
    ++fake_log.frees;
    g_held -= it->second.bytes;
    if (it->second.real) free(p);
    g_blocks.erase(it);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = calloc(n, 1); return hipSuccess; }
hipError_t hipHostFree(void *p) { free(p); return hipSuccess; }
hipError_t hipMemcpyAsync(void *dst, const void *src, size_t n, hipMemcpyKind kind, hipStream_t) {
    // (only small blocks hold anything)
    auto unreal = [](const void *p) { return (uintptr_t)p >= ((uintptr_t)1 << 44) && (char *)p < g_next; };
    if (!unreal(dst) && !unreal(src)) std::memcpy(dst, src, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = (hipEvent_t)calloc(1, 8); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 1.0f; return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = (hipStream_t)calloc(1, 8); return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *st) {
    *st = g_user_capture ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { ++g_own_capture; return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) {
    --g_own_capture;
    *g = (hipGraph_t)calloc(1, 8);
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t, hipGraphNode_t *, char *, size_t) {
    ++fake_log.graphs;
    *x = (hipGraphExec_t)calloc(1, 8);
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) { free(g); return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t x) { free(x); return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { ++fake_log.graph_launches; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) {
    std::memset(p, 0, sizeof(*p));
    std::strcpy(p->gcnArchName, "gfx950");
    p->multiProcessorCount = 256;
    return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *) {
    std::memset(a, 0, sizeof(*a));
    a->type = hipMemoryTypeDevice;
    return hipSuccess;
}
}

// ------------------------------------------------------------ launchers
namespace tess {
hipError_t launch_qsum(const LatticeParams &, const ViewParams &, double *, hipStream_t) { return launched(); }
hipError_t launch_setup(const LatticeParams &, const ViewParams &V, RecHead *, Payload *, DevCounters *, hipStream_t) {
    ++fake_log.setups;
    fake_log.edge_setups += V.edges ? 1 : 0;
    fake_log.stack_setups += V.nstack ? 1 : 0;
    fake_log.edges = V.edges;
    fake_log.nstack = V.nstack;
    fake_log.stored = (int64_t)V.own_cap;
    if (V.edges) fake_log.own_room = (int64_t)V.own_cap;
    fake_log.crease_bmax = V.crease_bmax;
    fake_log.bmax_per_q = V.bmax_per_q;
    return launched();
}
hipError_t launch_edges(const LatticeParams &, const ViewParams &, RecHead *, EdgePayload *, hipStream_t) { return launched(); }
hipError_t launch_count(const RecHead *, int64_t ntet, const BinParams &, uint32_t *, hipStream_t) {
    fake_log.ntet = ntet;
    return launched();
}
size_t scan_scratch_elems(int64_t n) { return (size_t)((n + 4095) / 4096) + 1; }
hipError_t launch_scan(const uint32_t *, uint64_t *, int64_t, uint64_t *, hipStream_t) { return launched(); }
hipError_t launch_totals(const uint32_t *, const uint64_t *, const BinParams &B, unsigned long long, PlanOut *out,
                         unsigned int *, hipStream_t) {
    out->total_pairs = g_pairs_per_tile * (unsigned long long)B.nbins;
    out->max_bin = g_pairs_per_tile;
    out->n_items = 0;
    out->own = B.edges ? g_own_count : 0;
    return launched();
}
hipError_t launch_plan(const uint32_t *, const uint64_t *, const BinParams &B, int32_t chunk, unsigned long long cap,
                       uint32_t *, PlanOut *, hipStream_t) {
    fake_log.Th = B.Th;
    fake_log.Tw = B.Tw;
    fake_log.chunk = chunk;
    fake_log.cap = cap;
    return launched();
}
hipError_t launch_items(const uint64_t *, const uint32_t *, const BinParams &, const PlanOut *, WorkItem *, hipStream_t) {
    return launched();
}
hipError_t launch_scatter(const RecHead *, int64_t, const BinParams &, const uint32_t *, const uint64_t *, uint32_t *,
                          unsigned long long, hipStream_t) {
    return launched();
}
hipError_t launch_zero(const ZeroList &, hipStream_t) { return launched(); }
hipError_t launch_raster(const RecHead *, const Payload *, const EdgePayload *, const uint32_t *, const WorkItem *,
                         uint64_t max_items, const PlanOut *, const BinParams &, int block, bool count, double *,
                         DevCounters *, hipStream_t) {
    ++fake_log.rasters;
    fake_log.counting_rasters += count ? 1 : 0;
    fake_log.block = block;
    fake_log.max_items = max_items;
    return launched();
}
hipError_t launch_raster_direct(const LatticeParams &, const ViewParams &, const RecHead *, const Payload *,
                                const EdgePayload *, const PlanOut *, unsigned long long, const BinParams &, double *,
                                DevCounters *, hipStream_t) {
    ++fake_log.direct_rasters;
    return launched();
}
hipError_t launch_stack_table(const double *, int, double *, hipStream_t) { return launched(); }
hipError_t launch_finalize(const double *, const BinParams &, float *, hipStream_t) { return launched(); }
hipError_t scratch_buffer(void **p) {
    // backed lazily by the system: only the plan slot is ever written
    static void *s = calloc(1, kScratchBytes);
    *p = s;
    return hipSuccess;
}
hipError_t launch_check_finite(const float *, const float *, const float *, int64_t, unsigned long long *, hipStream_t) {
    return launched();
}
hipError_t launch_scatter_ids(const float *, const float *, const float *, const uint64_t *, int64_t, float *, float *,
                              float *, unsigned int *, unsigned long long *, hipStream_t) {
    return launched();
}
}  // namespace tess
