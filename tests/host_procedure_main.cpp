// Driver of the whole per-layer procedure on a machine without a GPU: the few functions of the HIP runtime that the library calls are
// defined here (the program's own symbols take precedence over the runtime's), device memory is host memory and a kernel launch does nothing.  What is looked at
// is the host's part: what it allocates, what it waits for, and what it leaves behind when a step fails.  tests/test_procedure_host.py builds and runs it.
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "../include/sop.h"
#define float2 sop_kparams_float2          // (the HIP header has its own)
#include "../paper_2605_14929_amd/csrc/sop_kparams.h"
#undef float2

static int failures = 0;
#define CHECK(cond) do { if (!(cond)) { std::printf("CHECK failed line %d: %s\n", __LINE__, #cond); ++failures; } } while (0)

// ---- the stand-in runtime ----
static std::map<char*, size_t> g_device, g_pinned;
static std::string g_fail;                 // the next call of this function fails once
static int g_fail_after = 0;               // ... after so many that do not
static int g_searches_outside = 0;         // searches whose results would go to memory that nobody allocated
static int g_events = 0;                   // events alive
static bool g_capturing = false;           // the stream is being captured
static bool g_broken = false;              // ... and a call that no capture allows has been made (it ends the capture)
static std::string g_log;                  // waits ('e' event, 's' stream, 'd' device) and uploads from pinned memory ('u') in their order
static bool fails(const char* fn)
{
    if (g_fail != fn || g_fail_after-- > 0) return false;
    g_fail.clear();
    return true;
}
static void* take(std::map<char*, size_t>& of, size_t n)
{
    char* const p = static_cast<char*>(aligned_alloc(256, (n + 255) & ~size_t(255)));
    std::memset(p, 0, n);
    of[p] = n;
    return p;
}
static bool inside(const std::map<char*, size_t>& of, const void* q)
{
    for (const auto& b : of) if (q >= b.first && q < b.first + b.second) return true;
    return false;
}

extern "C" {
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int)
{
    std::memset(p, 0, sizeof(*p));
    p->multiProcessorCount = 256;
    p->sharedMemPerBlock = 160 * 1024;
    return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "stand-in error"; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) { *p = take(g_device, n); return hipSuccess; }
hipError_t hipFree(void* p) { CHECK(g_device.erase(static_cast<char*>(p)) == 1); free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned int) { if (g_capturing) { g_broken = true; return hipErrorStreamCaptureUnsupported; } if (fails("hipHostMalloc")) return hipErrorOutOfMemory; *p = take(g_pinned, n); return hipSuccess; }
hipError_t hipHostFree(void* p) { CHECK(g_pinned.erase(static_cast<char*>(p)) == 1); free(p); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned int) { if (fails("hipHostGetDevicePointer")) return hipErrorInvalidValue; *d = h; return hipSuccess; }
hipError_t hipMemset(void* p, int v, size_t n) { std::memset(p, v, n); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { if (inside(g_pinned, s)) g_log += 'u'; std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) { static char scratch[1 << 16]; *p = scratch; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 1; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned int) { if (fails("hipEventCreateWithFlags")) return hipErrorOutOfMemory; *e = reinterpret_cast<hipEvent_t>(new int(0)); ++g_events; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { delete reinterpret_cast<int*>(e); --g_events; return hipSuccess; }
// (an event recorded on a stream that is being captured stands for no work of the GPU: it can't be waited for)
hipError_t hipEventRecord(hipEvent_t e, hipStream_t)
{
    if (!e) return hipErrorInvalidHandle;
    if (fails("hipEventRecord")) return hipErrorOutOfMemory;
    *reinterpret_cast<int*>(e) = g_capturing;
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e)
{
    if (!e) return hipErrorInvalidHandle;
    if (*reinterpret_cast<int*>(e)) return hipErrorCapturedEvent;
    g_log += 'e';
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { if (g_capturing) { g_broken = true; return hipErrorStreamCaptureUnsupported; } g_log += 's'; return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { if (g_capturing) { g_broken = true; return hipErrorStreamCaptureUnsupported; } g_log += 'd'; return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) { *s = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* s, hipStream_t* st) { *g = *b = dim3(1, 1, 1); *s = 0; *st = nullptr; return hipSuccess; }
hipError_t hipLaunchKernel(const void*, dim3, dim3 block, void** args, size_t, hipStream_t)
{
    if (block.x >= 512) {                  // (a search: the calls made here launch no other kernel of so many threads)
        const KParams* p = static_cast<const KParams*>(args[0]);
        for (const double* out : {p->acos_pair, p->acos_atom})
            if (out && !inside(g_device, out) && !inside(g_pinned, out)) ++g_searches_outside;
    }
    return hipSuccess;
}
}

// ---- one call of the procedure: two codebooks, their pair ----
struct Layer {
    float nf[16], sh[16];
    sop_atom atoms[2];
    sop_layer_opts opts;
    sop_layer_result result;
    std::vector<char> room;
    char* ws = nullptr;
    size_t need = 0;
    sop_scale_fmt fmt;
    Layer(sop_ctx* c)
    {
        CHECK(sop_atom_nf(4, nf) == SOP_OK && sop_atom_sh(4, 1.5, -0.02, sh) == SOP_OK);
        atoms[0].n_entries = atoms[1].n_entries = 16;
        atoms[0].values = nf; atoms[1].values = sh;
        std::memset(&opts, 0, sizeof(opts));
        std::memset(&fmt, 0, sizeof(fmt));
        fmt.exp_bits = 4; fmt.man_bits = 3; fmt.bias = fmt.max_code = -1;
        CHECK(sop_search_layer_workspace(c, 256, 1024, 16, 2, &opts, &need) == SOP_OK);
        room.resize(need + 256);
        ws = reinterpret_cast<char*>((reinterpret_cast<uintptr_t>(room.data()) + 255) & ~uintptr_t(255));
    }
    sop_status call(sop_ctx* c, int shift = 0)
    {
        alignas(16) static char weights[16], norms[16];           // (never read: no kernel runs)
        return sop_search_layer(c, weights, SOP_BF16, 256, 1024, 1024, reinterpret_cast<float*>(norms), 16, fmt, shift, SOP_SEL_WSE, atoms, 2, &opts, ws, need,
                                &result, nullptr, nullptr, nullptr);
    }
};

// a step of the one-time set-up fails: the call says so, and the next one sets up again
static void setup_fails(const char* fn, int after)
{
    sop_ctx* c = nullptr;
    CHECK(sop_create(&c, 0) == SOP_OK);
    Layer l(c);
    const size_t pinned = g_pinned.size();
    const int events = g_events;
    g_fail = fn; g_fail_after = after;
    CHECK(l.call(c) == SOP_EHIP);
    CHECK(g_fail.empty());
    CHECK(g_pinned.size() == pinned && g_events == events);      // (nothing half set up)
    CHECK(l.call(c) == SOP_OK && l.result.kind == 0);
    CHECK(l.call(c) == SOP_OK);
    CHECK(g_searches_outside == 0);
    CHECK(sop_destroy(c) == SOP_OK);
    CHECK(g_pinned.empty() && g_device.empty() && g_events == 0);
}

// no event could be recorded behind a call's work: the call says so where nothing else went wrong, and the next one waits for all of it before it writes to the staging buffers
static void record_fails(bool call_fails)
{
    sop_ctx* c = nullptr;
    CHECK(sop_create(&c, 0) == SOP_OK);
    Layer l(c);
    CHECK(l.call(c) == SOP_OK);
    g_fail = "hipEventRecord"; g_fail_after = 0;
    CHECK(l.call(c, call_fails ? 100 : 0) == (call_fails ? SOP_EFMT : SOP_EHIP));
    CHECK(g_fail.empty());
    g_log.clear();
    CHECK(l.call(c) == SOP_OK);
    CHECK(g_log[0] == 'd');
    g_log.clear();
    CHECK(l.call(c) == SOP_OK);
    CHECK(g_log[0] == 'e');
    CHECK(sop_destroy(c) == SOP_OK);
}

// a call on a stream that is being captured is refused, whatever else is wrong with it and also as a context's first, and leaves capture and context as they were
static void captured(int shift, bool first)
{
    sop_ctx* c = nullptr;
    CHECK(sop_create(&c, 0) == SOP_OK);
    Layer l(c);
    if (!first) CHECK(l.call(c) == SOP_OK);
    g_capturing = true;
    CHECK(l.call(c, shift) != SOP_OK);
    CHECK(!g_broken);
    g_capturing = false;
    CHECK(l.call(c) == SOP_OK);
    CHECK(l.call(c) == SOP_OK);
    CHECK(sop_destroy(c) == SOP_OK);
}

int main(int argc, char** argv)
{
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "setup") setup_fails(argv[2], std::atoi(argv[3]));
    else if (what == "record") record_fails(std::atoi(argv[2]) != 0);
    else if (what == "captured") captured(std::atoi(argv[2]), std::atoi(argv[3]) != 0);
    else { std::printf("usage: %s setup FUNCTION CALLS_BEFORE | record CALL_FAILS | captured SHIFT FIRST\n", argv[0]); return 2; }
    if (failures) return 1;
    std::printf("procedure ok\n");
    return 0;
}
