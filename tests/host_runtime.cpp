// host_runtime.cpp -- a stand-in for the HIP runtime, linked with the library's
// host code (compiled without its kernels) so that the host side can be tested
// without a GPU: device memory is host memory, copies are memcpy, and a launch is
// only recorded, with the dynamic LDS it asks for and the limit its function has
// at that moment.  Streams have clocks: a launch takes a millisecond, waiting for an
// event a second, and events hold their stream's time.  A launch of the sweep marks every sample of its queue as done.
// Allocations of the host code are counted and can be made to fail.
#include <hip/hip_runtime.h>
#include <malloc.h>

#include <atomic>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "../paper_2607_18991_amd/csrc/nz_internal.h"

#define FAKE extern "C" __attribute__((visibility("default")))

namespace {
struct Launch {
    std::string name;
    size_t lds, limit;
    hipStream_t stream;
};
std::mutex g_lock;
// (kernels are registered before this file's globals are constructed)
std::map<const void *, std::string> &names()
{
    static std::map<const void *, std::string> m;
    return m;
}
std::map<const void *, size_t> g_limits;
std::map<void *, size_t> g_blocks;
std::map<hipStream_t, float> g_clock;
std::map<hipEvent_t, float> g_events;
std::vector<Launch> g_launches;
int64_t g_mallocs = 0, g_frees = 0, g_streams = 0;
void *g_bad_stream = nullptr;   // copies on it fail
bool g_bad_copies = false;
int g_bad_mallocs = 0;          // so many allocations of device memory fail
// host allocations of the calling thread: bytes held and their peak, and the
// number of allocations until one fails (< 0: none)
thread_local int64_t t_held = 0, t_peak = 0, t_left = -1;
thread_local hipStream_t t_stream;
thread_local dim3 t_grid, t_block;
thread_local size_t t_lds;

// (malloc and free without a header: the C++ library's own code allocates and
// frees some of the same objects)
void *take(size_t n)
{
    if (t_left == 0) throw std::bad_alloc();
    if (t_left > 0) --t_left;
    void *p = std::malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    t_held += static_cast<int64_t>(malloc_usable_size(p));
    if (t_held > t_peak) t_peak = t_held;
    return p;
}
void give(void *p)
{
    if (p) t_held -= static_cast<int64_t>(malloc_usable_size(p));
    std::free(p);
}
}  // namespace

void *operator new(size_t n) { return take(n); }
void *operator new[](size_t n) { return take(n); }
void operator delete(void *p) noexcept { give(p); }
void operator delete[](void *p) noexcept { give(p); }
void operator delete(void *p, size_t) noexcept { give(p); }
void operator delete[](void *p, size_t) noexcept { give(p); }

// ---- what the tests set and read
FAKE void fake_reset()
{
    std::lock_guard<std::mutex> g(g_lock);
    g_launches.clear();
    g_mallocs = g_frees = 0;
    g_bad_copies = false;
}
FAKE int fake_launches() { return static_cast<int>(g_launches.size()); }
FAKE const char *fake_launch(int k, size_t *lds, size_t *limit)
{
    *lds = g_launches[k].lds;
    *limit = g_launches[k].limit;
    return g_launches[k].name.c_str();
}
FAKE void *fake_launch_stream(int k) { return g_launches[k].stream; }
FAKE int64_t fake_mallocs() { return g_mallocs; }
FAKE int64_t fake_frees() { return g_frees; }
FAKE int64_t fake_device_bytes()
{
    std::lock_guard<std::mutex> g(g_lock);
    int64_t sum = 0;
    for (const auto &b : g_blocks) sum += static_cast<int64_t>(b.second);
    return sum;
}
FAKE void fake_fail_copies(void *stream)
{
    g_bad_stream = stream;
    g_bad_copies = true;
}
FAKE void fake_fail_mallocs(int n) { g_bad_mallocs = n; }
FAKE void fake_fail_new(int64_t after) { t_left = after; }
FAKE void fake_reset_peak() { t_held = t_peak = 0; }
FAKE int64_t fake_peak() { return t_peak; }

// ---- the runtime
FAKE void **__hipRegisterFatBinary(const void *) { return nullptr; }
FAKE void __hipUnregisterFatBinary(void **) {}
FAKE void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned, void *, void *, void *, void *, int *)
{
    names()[f] = name;
}
FAKE void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
FAKE hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t st)
{
    t_grid = grid;
    t_block = block;
    t_lds = lds;
    t_stream = st;
    return hipSuccess;
}
FAKE hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *st)
{
    *grid = t_grid;
    *block = t_block;
    *lds = t_lds;
    *st = t_stream;
    return hipSuccess;
}
FAKE hipError_t hipLaunchKernel(const void *f, dim3, dim3, void **args, size_t lds, hipStream_t st)
{
    std::lock_guard<std::mutex> g(g_lock);
    const std::string &name = names()[f];
    const auto it = g_limits.find(f);
    g_clock[st] += 1.0f;
    g_launches.push_back({name, lds, it == g_limits.end() ? 65536 : it->second, st});
    if (name.find("nz_sweep_kernel") != std::string::npos) {
        const NzSweepArgs &a = *static_cast<const NzSweepArgs *>(args[0]);
        for (int32_t k = 0; k < a.nqueue; ++k) a.state[k].status = NZ_ST_DONE;
    }
    return hipSuccess;
}
FAKE hipError_t hipFuncSetAttribute(const void *f, hipFuncAttribute, int value)
{
    std::lock_guard<std::mutex> g(g_lock);
    g_limits[f] = static_cast<size_t>(value);
    return hipSuccess;
}
FAKE hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t)
{
    *n = 1;
    return hipSuccess;
}
FAKE hipError_t hipGetLastError() { return hipSuccess; }
FAKE const char *hipGetErrorString(hipError_t) { return "stand-in error"; }
FAKE hipError_t hipGetDevice(int *id)
{
    *id = 0;
    return hipSuccess;
}
FAKE hipError_t hipSetDevice(int) { return hipSuccess; }
FAKE hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int)   // (a macro of the versioned name)
{
    std::memset(p, 0, sizeof *p);
    p->multiProcessorCount = 256;
    p->sharedMemPerBlock = 65536;
    return hipSuccess;
}
FAKE hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int)
{
    *v = 163840;
    return hipSuccess;
}
FAKE hipError_t hipMemGetInfo(size_t *freeb, size_t *total)
{
    *freeb = size_t(64) << 30;
    *total = size_t(288) << 30;
    return hipSuccess;
}
FAKE hipError_t hipMalloc(void **p, size_t n)
{
    std::lock_guard<std::mutex> g(g_lock);
    if (g_bad_mallocs > 0) {
        --g_bad_mallocs;
        return hipErrorOutOfMemory;
    }
    *p = std::calloc(1, n);   // (pages come when they are touched)
    g_blocks[*p] = n;
    ++g_mallocs;
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
FAKE hipError_t hipFree(void *p)
{
    if (!p) return hipSuccess;
    std::lock_guard<std::mutex> g(g_lock);
    g_blocks.erase(p);
    ++g_frees;
    std::free(p);
    return hipSuccess;
}
static hipError_t copy(void *d, const void *s, size_t n, hipStream_t st)
{
    if (g_bad_copies && st == g_bad_stream) return hipErrorInvalidValue;
    std::memcpy(d, s, n);
    return hipSuccess;
}
FAKE hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t st) { return copy(d, s, n, st); }
FAKE hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { return copy(d, s, n, nullptr); }
FAKE hipError_t hipMemset(void *d, int v, size_t n)
{
    std::memset(d, v, n);
    return hipSuccess;
}
FAKE hipError_t hipGetSymbolAddress(void **p, const void *)
{
    static void *block = std::aligned_alloc(4096, size_t(256) << 20);   // (the one symbol: the static buffer)
    *p = block;
    return hipSuccess;
}
FAKE hipError_t hipStreamCreateWithFlags(hipStream_t *st, unsigned)
{
    *st = reinterpret_cast<hipStream_t>(static_cast<uintptr_t>(0x1000 + ++g_streams));
    return hipSuccess;
}
FAKE hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
FAKE hipError_t hipStreamWaitEvent(hipStream_t st, hipEvent_t, unsigned)
{
    std::lock_guard<std::mutex> g(g_lock);
    g_clock[st] += 1000.0f;
    return hipSuccess;
}
FAKE hipError_t hipEventCreate(hipEvent_t *e)
{
    static std::atomic<uintptr_t> next{0x2000};
    *e = reinterpret_cast<hipEvent_t>(next++);
    return hipSuccess;
}
FAKE hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
FAKE hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
FAKE hipError_t hipEventRecord(hipEvent_t e, hipStream_t st)
{
    std::lock_guard<std::mutex> g(g_lock);
    g_events[e] = g_clock[st];
    return hipSuccess;
}
FAKE hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
FAKE hipError_t hipEventElapsedTime(float *ms, hipEvent_t a, hipEvent_t b)
{
    std::lock_guard<std::mutex> g(g_lock);
    *ms = g_events[b] - g_events[a];
    return hipSuccess;
}
