// The library's host source on top of a runtime that lives in host memory and launchers that write down what they are
// asked to launch: which kernels a call issues, with how many units, can then be tested without a GPU.  Built and
// loaded by test_launch_routes.py; "device" pointers are host addresses, and no kernel runs.
#include "lora_internal.h"
#include <cstdlib>
#include <cstring>
#include <string>

static std::string g_log, g_forms;
static int g_capturing, g_big_spread, g_walks;
static struct Memory { uintptr_t from; size_t bytes; hipMemoryType type; } g_memory[8];  // what this runtime knows of, besides what it gave out
static int g_n_memory;

static hipError_t note(const std::string &s)
{
    g_log += s + "\n";
    return hipSuccess;
}
// of a launcher that chooses between kernels, the one it takes
static void form(const char *s) { g_forms += std::string(s) + " "; }
static std::string num(long long v) { return " " + std::to_string(v); }

extern "C" {
const char *recorder_take()
{
    static std::string out;
    out.swap(g_log);
    g_log.clear();
    return out.c_str();
}
const char *recorder_take_forms()
{
    static std::string out;
    out.swap(g_forms);
    g_forms.clear();
    return out.c_str();
}
// whether the last launch of 64-token expand units asked for three work groups per compute unit
int recorder_big_spread() { return g_big_spread; }
// ... and how many strips of their unit its work groups walk (0: they take 256 columns)
int recorder_walks() { return g_walks; }
// 1: the stream captures; 2: it is the legacy stream and a blocking stream captures
void recorder_capture(int on) { g_capturing = on; }

// memory of a caller's as this runtime knows it: an allocation of pinned host memory, or of the device's
void recorder_memory(void *p, size_t bytes, int pinned)
{
    g_memory[g_n_memory++ % 8] = {(uintptr_t)p, bytes, pinned ? hipMemoryTypeHost : hipMemoryTypeDevice};
}
static const Memory *known(const void *p)
{
    for (const Memory &m : g_memory)
        if ((uintptr_t)p >= m.from && (uintptr_t)p - m.from < m.bytes) return &m;
    return nullptr;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *at, const void *p)
{
    const Memory *m = known(p);
    if (!m) return hipErrorInvalidValue;
    memset(at, 0, sizeof *at);
    at->type = m->type;
    at->devicePointer = const_cast<void *>(p);
    return hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t *base, size_t *bytes, hipDeviceptr_t p)
{
    const Memory *m = known(p);
    if (!m) return hipErrorNotFound;
    *base = (hipDeviceptr_t)m->from;
    *bytes = m->bytes;
    return hipSuccess;
}

hipError_t hipMalloc(void **p, size_t n) { return (*p = aligned_alloc(4096, (n + 4095) / 4096 * 4096)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void *p) { free(p); return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipHostFree(void *p) { return hipFree(p); }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { memmove(d, s, n); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = (hipEvent_t)malloc(1); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { free(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = (hipStream_t)malloc(1); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { free(s); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s)
{
    *s = g_capturing == 1 ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return g_capturing == 2 ? hipErrorStreamCaptureImplicit : hipSuccess;
}
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int)
{
    memset(p, 0, sizeof *p);
    strcpy(p->gcnArchName, "gfx950");
    p->multiProcessorCount = 256;
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "error"; }
}

namespace lora {
static void slices_form(const SyncArgs *sync) { form(!sync ? "callers" : sync->parts ? "by_expand" : "by_shrink"); }
hipError_t launch_shrink(const LaunchCtx &c, const uint16_t *, int64_t, int, float *, int, int64_t, const SyncArgs *sync, hipStream_t)
{
    if (!c.n_units) return hipSuccess;
    slices_form(sync);
    return note("shrink" + num(c.n_units));
}
hipError_t launch_shrink_wide(const LaunchCtx &c, bool, const uint16_t *, int64_t, int, int, float *, uint16_t *, uint16_t *, hipStream_t) { return c.n_units ? note("shrink_wide" + num(c.n_units)) : hipSuccess; }
hipError_t launch_expand(const LaunchCtx &c, bool big, const float *, uint16_t *, int64_t, const SyncArgs *sync, hipStream_t)
{
    if (!c.n_units) return hipSuccess;
    if (!big) slices_form(sync);
    else g_big_spread = big_spread(c), g_walks = !sync && expand_walks(c) ? walk_strips(c) : 0;
    return note((big ? "expand_big" : "expand") + num(c.n_units));
}
hipError_t launch_shrink_prefill(const LaunchCtx &c, int, const uint16_t *, int64_t, uint16_t *, uint16_t *, float *, int n_slices, int64_t, float *, const SyncArgs *, hipStream_t)
{
    if (!c.n_units) return hipSuccess;
    form(shrink_in_halves(c) ? "halves" : "whole");
    return note("shrink_prefill" + num(c.n_units) + num(n_slices));
}
hipError_t launch_shrink_mixed(const LaunchCtx &h, int, const LaunchCtx &c, const uint16_t *, int64_t, int, float *, int, int64_t, const SyncArgs *sync, hipStream_t)
{
    slices_form(sync);
    return note("shrink_mixed" + num(h.n_units) + num(c.n_units));
}
hipError_t launch_expand_mixed(const LaunchCtx &b, const LaunchCtx &c, uint16_t *, int64_t, const SyncArgs *sync, hipStream_t)
{
    slices_form(sync);
    return note("expand_mixed" + num(b.n_units) + num(c.n_units));
}
hipError_t launch_apply_fused(const LaunchCtx &s, const LaunchCtx &e, const uint16_t *, int64_t, int, float *, int, int64_t, uint16_t *, int64_t, const SyncArgs *, hipStream_t) { return note("apply_fused" + num(s.n_units) + num(e.n_units)); }
hipError_t launch_decode_fused(const LaunchCtx &, const LaunchCtx &, int grid, const uint16_t *, int64_t, int, int, uint16_t *, int64_t, unsigned, const SyncArgs *, hipStream_t) { return note("decode_fused" + num(grid)); }
hipError_t launch_reduce_slices(const float *, int n, int64_t, float *, int64_t, hipStream_t) { return note("reduce_slices" + num(n)); }
hipError_t launch_copy_in(const void *a, size_t a_bytes, const void *b, size_t b_bytes, void *dev, hipStream_t)
{
    memmove(dev, a, a_bytes);
    if (b_bytes) memmove((char *)dev + a_bytes, b, b_bytes);
    return note("copy_in" + num((long long)a_bytes) + num((long long)b_bytes));
}
hipError_t launch_pack_adapter(const uint16_t *, const uint16_t *, int, int, int, int, uint16_t *, uint16_t *, hipStream_t) { return hipSuccess; }
hipError_t launch_linear_lora(const int32_t *, const LinBlock *b, int n_places, const uint16_t *, const uint16_t *, const uint16_t *, int64_t, int, int out, const uint16_t *, const uint16_t *, uint16_t *, int64_t, hipStream_t)
{
    if (b->big_tiles == 0) {
        const LinSmallTiles t = linear_small_tiles(n_places, out);
        g_forms += std::to_string(16 * t.rb) + "x" + std::to_string(16 * t.cb) + (t.pairs() ? "_in_pairs " : " ");
    }
    return note("linear" + num(n_places) + num(b->big_tiles));
}
hipError_t launch_pack_weight(const uint16_t *, int, int, uint16_t *, hipStream_t) { return hipSuccess; }
hipError_t probe_xcc(unsigned *x, int n, hipStream_t)
{
    for (int b = 0; b < n; ++b) x[b] = (unsigned)b % 8;
    return hipSuccess;
}
hipError_t static_scratch(void **p)
{
    static char *mem = (char *)aligned_alloc(4096, kStaticScratchBytes);
    *p = mem;
    return hipSuccess;
}
}
