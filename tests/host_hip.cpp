// A HIP runtime for tests of the library's host code on a machine without a GPU.
// Allocations come from the C heap and can be made to fail, launches are recorded
// with their kernel's name and do nothing, and the last error is kept the way HIP
// keeps it: a failed call sets it, only hipGetLastError clears it, later successes
// leave it alone.
#include <hip/hip_runtime_api.h>

#include <cxxabi.h>

#include <cstdlib>
#include <map>
#include <string>

namespace {

hipError_t last_error = hipSuccess;
size_t malloc_limit = ~(size_t)0;  // larger requests fail
long live = 0;                     // allocations not freed yet
bool sync_fails = false;           // as under stream capture
std::string launches;
dim3 cfg_grid, cfg_block;
size_t cfg_lds;
hipStream_t cfg_stream;

hipError_t fail(hipError_t e) { return last_error = e; }

// kernels register before this file's own constructors run
std::map<const void *, std::string> &names()
{
    static std::map<const void *, std::string> m;
    return m;
}

}  // namespace

extern "C" {

void host_hip_set_malloc_limit(size_t bytes) { malloc_limit = bytes; }
void host_hip_set_sync_fails(int fails) { sync_fails = fails != 0; }
long host_hip_live_allocations(void) { return live; }
void host_hip_clear_launches(void) { launches.clear(); }
// one line per launch: kernel<template arguments> grid.x grid.y block.x dynamic LDS bytes
const char *host_hip_launches(void) { return launches.c_str(); }

hipError_t hipMalloc(void **p, size_t n)
{
    *p = nullptr;
    if (n > malloc_limit || !(*p = std::calloc(n, 1)))
        return fail(hipErrorOutOfMemory);
    ++live;
    return hipSuccess;
}

hipError_t hipFree(void *p)
{
    live -= p != nullptr;
    std::free(p);
    return hipSuccess;
}

hipError_t hipGetLastError(void)
{
    const hipError_t e = last_error;
    last_error = hipSuccess;
    return e;
}

hipError_t hipGetDevice(int *d)
{
    *d = 0;
    return hipSuccess;
}

hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t)
{
    return sync_fails ? fail(hipErrorStreamCaptureUnsupported) : hipSuccess;
}
hipError_t hipMemcpyAsync(void *, const void *, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }

hipError_t hipGetSymbolAddress(void **p, const void *)
{
    static char symbol[256];
    *p = symbol;
    return hipSuccess;
}

hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t s)
{
    cfg_grid = grid, cfg_block = block, cfg_lds = lds, cfg_stream = s;
    return hipSuccess;
}

hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *s)
{
    *grid = cfg_grid, *block = cfg_block, *lds = cfg_lds, *s = cfg_stream;
    return hipSuccess;
}

hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **, size_t lds, hipStream_t)
{
    launches += names()[f] + " " + std::to_string(grid.x) + " " + std::to_string(grid.y) + " " +
                std::to_string(block.x) + " " + std::to_string(lds) + "\n";
    return hipSuccess;
}

void **__hipRegisterFatBinary(const void *)
{
    static void *handle;
    return &handle;
}

void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}

void __hipRegisterFunction(void **, const void *host, char *, const char *device, unsigned, void *,
                           void *, void *, void *, int *)
{
    int st = 0;
    char *d = abi::__cxa_demangle(device, nullptr, nullptr, &st);
    std::string s = st == 0 ? d : device;
    std::free(d);
    for (const char *cut : {"void ", "cdk::", "(anonymous namespace)::"})
        for (size_t at; (at = s.find(cut)) != std::string::npos;)
            s.erase(at, std::string(cut).size());
    s = s.substr(0, s.find('('));  // the name and its template arguments
    for (size_t at; (at = s.find(' ')) != std::string::npos;)
        s.erase(at, 1);
    names()[host] = s;
}

}  // extern "C"
