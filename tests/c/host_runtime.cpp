// host_runtime.cpp -- a HIP runtime without a GPU, for tests of the library's
// host code: device memory is host memory (with a limit that allocations run
// into), copies and fills happen at once, and a kernel launch calls a hook with
// the kernel's name and arguments, which plays the kernel's part.
//
// Linked with the library's own objects into a library that is loaded by itself.
#include <hip/hip_runtime_api.h>

#include <sys/mman.h>

#include <cstdio>
#include <cstring>
#include <map>
#include <string>

namespace {

typedef void (*Hook)(const char *name, void **args, unsigned grid, unsigned block);

Hook g_hook = nullptr;
std::map<const void *, std::string> g_names;
std::map<void *, size_t> g_allocs;
size_t g_used = 0, g_limit = ~(size_t)0, g_refused = 0;
constexpr size_t kMoved = 64u << 20;  // larger copies and fills are left out: the memory behind them is never touched
dim3 g_grid, g_block;
size_t g_shared = 0;
hipStream_t g_stream = nullptr;
unsigned char g_symbol[1 << 20];

}  // namespace

extern "C" {

// ---- for the tests ----
void host_runtime_hook(Hook h) { g_hook = h; }
void host_runtime_limit(size_t bytes) { g_limit = bytes; }
size_t host_runtime_used(void) { return g_used; }
size_t host_runtime_refused(void) { return g_refused; }

// ---- what compiled host code registers and launches with ----
void **__hipRegisterFatBinary(const void *) {
    static void *handle = nullptr;
    return &handle;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, uint3 *, uint3 *, dim3 *,
                           dim3 *, int *) {
    g_names[host] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t s) {
    g_grid = grid;
    g_block = block;
    g_shared = shared;
    g_stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shared, hipStream_t *s) {
    *grid = g_grid;
    *block = g_block;
    *shared = g_shared;
    *s = g_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t, hipStream_t) {
    const auto it = g_names.find(f);
    if (g_hook) g_hook(it == g_names.end() ? "?" : it->second.c_str(), args, grid.x, block.x);
    return hipSuccess;
}

// ---- memory ----
hipError_t hipMalloc(void **p, size_t n) {
    *p = nullptr;
    n = n ? n : 1;
    if (g_used + n > g_limit) {
        g_refused++;
        return hipErrorOutOfMemory;
    }
    void *m = mmap(nullptr, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (m == MAP_FAILED) return hipErrorOutOfMemory;
    g_allocs[m] = n;
    g_used += n;
    *p = m;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    if (!p) return hipSuccess;
    const auto it = g_allocs.find(p);
    if (it == g_allocs.end()) {
        std::fprintf(stderr, "hipFree of memory that is not allocated\n");
        return hipErrorInvalidValue;
    }
    munmap(p, it->second);
    g_used -= it->second;
    g_allocs.erase(it);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
    *p = calloc(1, n);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipHostFree(void *p) {
    free(p);
    return hipSuccess;
}
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned) {
    *d = h;
    return hipSuccess;
}
// Whether [p, p + n) lies in one allocation, or in none (host memory).
static bool inside(const void *p, size_t n) {
    auto it = g_allocs.upper_bound(const_cast<void *>(p));
    if (it == g_allocs.begin()) return true;
    --it;
    const char *end = (const char *)it->first + it->second;
    return (const char *)p >= end || (const char *)p + n <= end;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
    if (!inside(d, n) || !inside(s, n)) return hipErrorInvalidValue;
    if (n <= kMoved) std::memmove(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t) { return hipMemcpy(d, s, n, k); }
hipError_t hipMemset(void *d, int v, size_t n) {
    if (!inside(d, n)) return hipErrorInvalidValue;
    if (n <= kMoved) std::memset(d, v, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { return hipMemset(d, v, n); }
hipError_t hipGetSymbolAddress(void **p, const void *) {
    *p = g_symbol;
    return hipSuccess;
}

// ---- device, streams, events ----
hipError_t hipGetDevice(int *d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) {
    *v = 64;
    return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) {
    std::memset(p, 0, sizeof(*p));
    std::strcpy(p->gcnArchName, "gfx950");
    p->warpSize = 64;
    p->multiProcessorCount = 256;
    return hipSuccess;
}
int hipGetStreamDeviceId(hipStream_t) { return 0; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) {
    *s = hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
    *e = nullptr;
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }

}  // extern "C"
