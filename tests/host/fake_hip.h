// A HIP runtime for the library's host code on a machine without a device.
// Device memory is mapped host memory that is never given out twice; a free or
// a copy that does not lie in a live allocation is a fault; kernels are
// counted by name and not run.  The functions here take the place of the HIP
// runtime's for an executable that includes this file and links the library.
#pragma once

#include <hip/hip_runtime_api.h>
#include <sys/mman.h>

#include <cstdint>
#include <cstdio>
#include <cstring>
#include <functional>
#include <map>
#include <string>

namespace fake {

struct Runtime {
    std::map<uintptr_t, size_t> live;              // allocations by address
    std::map<const void *, std::string> names;     // kernels by their host stub
    std::map<std::string, int> launches;           // by (mangled) name
    size_t limit = SIZE_MAX;                       // largest allocation granted
    size_t largest = 0;                            // and asked for
    int mallocs = 0, frees = 0, refused = 0, syncs = 0, faults = 0;
    bool capturing = false;                        // every stream
    std::function<bool(void *, size_t)> read;      // fills a copy to the host in the kernels' place, if it knows it
};

inline Runtime &rt()
{
    static Runtime *r = new Runtime();  // kernels are registered before main
    return *r;
}

inline void fault(const char *what, const void *p)
{
    ++rt().faults;
    std::printf("fault: %s %p\n", what, p);
}

inline bool inside(const void *p, size_t n)
{
    auto it = rt().live.upper_bound((uintptr_t)p);
    return it != rt().live.begin() && (--it, (uintptr_t)p + n <= it->first + it->second);
}

// Launches of the kernels whose name holds `part`.
inline int launches(const char *part)
{
    int n = 0;
    for (const auto &k : rt().launches)
        if (k.first.find(part) != std::string::npos) n += k.second;
    return n;
}

}  // namespace fake

extern "C" {

void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, dim3 *,
                           dim3 *, int *)
{
    fake::rt().names[host] = name;
}
void **__hipRegisterFatBinary(const void *)
{
    static void *handle;
    return &handle;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void **) {}

static struct {
    dim3 grid, block;
    size_t lds;
    hipStream_t st;
} g_config;
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t st)
{
    g_config = {grid, block, lds, st};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *st)
{
    *grid = g_config.grid;
    *block = g_config.block;
    *lds = g_config.lds;
    *st = g_config.st;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **, size_t, hipStream_t)
{
    const std::string &name = fake::rt().names[f];
    if (grid.x == 0 || grid.y == 0 || grid.y > 65535 || block.x == 0 || (uint64_t)grid.x * block.x >= (1ull << 32)) {
        std::printf("fault: %s on %u x %u blocks of %u\n", name.c_str(), grid.x, grid.y, block.x);
        ++fake::rt().faults;
    }
    ++fake::rt().launches[name];
    return hipSuccess;
}

hipError_t hipMalloc(void **p, size_t n)
{
    fake::Runtime &r = fake::rt();
    *p = nullptr;
    if (r.capturing) fake::fault("allocation under capture", nullptr);
    r.largest = n > r.largest ? n : r.largest;
    if (n > r.limit) {
        ++r.refused;
        return hipErrorOutOfMemory;
    }
    const size_t len = (n + 4095) / 4096 * 4096 + 4096;
    void *m = mmap(nullptr, len, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (m == MAP_FAILED) return hipErrorOutOfMemory;
    r.live[(uintptr_t)m] = n;
    ++r.mallocs;
    *p = m;
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    fake::Runtime &r = fake::rt();
    if (!p) return hipSuccess;
    auto it = r.live.find((uintptr_t)p);
    if (r.capturing) fake::fault("free under capture", p);
    if (it == r.live.end()) {
        fake::fault("free of memory that is not allocated:", p);
        return hipErrorInvalidValue;
    }
    const size_t len = (it->second + 4095) / 4096 * 4096 + 4096;
    mmap(p, len, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE | MAP_FIXED, -1, 0);  // never reused
    r.live.erase(it);
    ++r.frees;
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind kind)
{
    fake::Runtime &r = fake::rt();
    if (kind != hipMemcpyDeviceToHost && !fake::inside(d, n)) {
        fake::fault("copy to memory that is not allocated:", d);
        return hipErrorInvalidValue;
    }
    if (kind != hipMemcpyHostToDevice && !fake::inside(s, n)) {
        fake::fault("copy from memory that is not allocated:", s);
        return hipErrorInvalidValue;
    }
    if (!(kind == hipMemcpyDeviceToHost && r.read && r.read(d, n))) std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind kind, hipStream_t) { return hipMemcpy(d, s, n, kind); }
hipError_t hipMemset(void *p, int v, size_t n)
{
    if (!fake::inside(p, n)) {
        fake::fault("clearing of memory that is not allocated:", p);
        return hipErrorInvalidValue;
    }
    std::memset(p, v, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *p, int v, size_t n, hipStream_t) { return hipMemset(p, v, n); }

hipError_t hipStreamSynchronize(hipStream_t)
{
    ++fake::rt().syncs;
    if (fake::rt().capturing) fake::fault("synchronisation under capture", nullptr);
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s)
{
    *s = fake::rt().capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "error of the fake runtime"; }
hipError_t hipGetDeviceCount(int *n)
{
    *n = 1;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int)
{
    *v = 256;  // asked for the compute units
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t)
{
    *n = 8;
    return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p)
{
    std::memset(a, 0, sizeof(*a));
    a->type = fake::inside(p, 1) ? hipMemoryTypeDevice : hipMemoryTypeHost;
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *)
{
    static void *array = mmap(nullptr, 64u << 20, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    *p = array;
    return hipSuccess;
}

}  // extern "C"
