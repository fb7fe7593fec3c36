// A stand-in for the HIP runtime that the library's host code runs over on a
// CPU: no kernel runs, device memory is host memory, the launch of a given
// number fails, and the grids are seen.  (Included by a program that loads the
// library and exports its own symbols.)
#pragma once

#include <hip/hip_runtime_api.h>
#include <stdlib.h>
#include <string.h>

#include "wcnst.h"

static int launches = 0, fail_at = 0;
static unsigned long long last_groups = 0;  // workgroups of the last launch
static hipError_t last = hipSuccess;
static dim3 cfg_grid, cfg_block;
static size_t cfg_shared;
static hipStream_t cfg_stream;

static void* cells(size_t n)
{
    void* p = aligned_alloc(256, (n + 255) / 256 * 256);
    if (!p) abort();
    return memset(p, 0, n);
}

extern "C" {
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t n, hipStream_t s)
{
    cfg_grid = g;
    cfg_block = b;
    cfg_shared = n;
    cfg_stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* n, hipStream_t* s)
{
    *g = cfg_grid;
    *b = cfg_block;
    *n = cfg_shared;
    *s = cfg_stream;
    return hipSuccess;
}
void** __hipRegisterFatBinary(const void*)
{
    static void* handle;
    return &handle;
}
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void**) {}
hipError_t hipLaunchKernel(const void*, dim3 g, dim3, void**, size_t, hipStream_t)
{
    last_groups = (unsigned long long)g.x * g.y * g.z;
    if (++launches != fail_at) return hipSuccess;
    return last = hipErrorOutOfMemory;
}
hipError_t hipGetLastError(void)
{
    const hipError_t e = last;
    last = hipSuccess;
    return e;
}
const char* hipGetErrorString(hipError_t) { return "stand-in"; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned)
{
    *p = cells(n);
    return hipSuccess;
}
hipError_t hipHostFree(void* p)
{
    free(p);
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned)
{
    *e = nullptr;
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t)
{
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind)
{
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipGetDevice(int* d)
{
    *d = 0;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int)
{
    *v = 256;
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*)
{
    static void* scratch = cells(WCNST_NOALLOC_MAX_BYTES);
    *p = scratch;
    return hipSuccess;
}
}
