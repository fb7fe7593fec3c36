// Whether an entry point reports a kernel launch that fails: the library over
// a stand-in for the HIP runtime, in which no kernel runs, device memory is
// host memory, and the launch of a given number fails.
//
// wcnst_launchcheck LIB ENTRY NDIM NX: for n = 1, 2, ... prints the status of
// the entry point when its n-th launch fails, then that of a call without a
// failure (for an n beyond its launches), on a line.
#include <dlfcn.h>
#include <hip/hip_runtime_api.h>
#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include "wcnst.h"

static int launches = 0, fail_at = 0;
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
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t)
{
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

#define SYM(name) auto* name##_ = reinterpret_cast<decltype(&name)>(dlsym(so, #name))

int main(int argc, char** argv)
{
    void* so = argc == 5 ? dlopen(argv[1], RTLD_NOW) : nullptr;
    if (!so) return 2;
    SYM(wcnst_desc_init);
    SYM(wcnst_workspace_size);
    SYM(wcnst_create);
    SYM(wcnst_step);
    SYM(wcnst_solve);
    SYM(wcnst_solve_noalloc);
    SYM(wcnst_rhs);
    SYM(wcnst_destroy);
    const char* entry = argv[2];
    wcnst_desc d;
    if (wcnst_desc_init_(&d)) return 3;
    d.ndim = atoi(argv[3]);
    d.nx = atoi(argv[4]);
    d.ny = d.ndim == 2 ? d.nx : 1;
    size_t bytes = 0;
    if (wcnst_workspace_size_(&d, &bytes)) return 3;
    const size_t n = sizeof(double) * 4 * (size_t)d.nx * (size_t)d.ny;
    void* ws = cells(bytes);
    double *U = (double*)cells(n), *R = (double*)cells(n);
    for (int k = 1;; ++k) {
        wcnst_solver* s = nullptr;
        fail_at = 0;
        if (wcnst_create_(&d, nullptr, ws, bytes, &s)) return 4;
        launches = 0;
        fail_at = k;
        int st = -1;
        if (!strcmp(entry, "step")) st = wcnst_step_(s, U, 0.0, 0.5);
        if (!strcmp(entry, "step_dt")) st = wcnst_step_(s, U, 0.1, 0.0);
        if (!strcmp(entry, "rhs")) st = wcnst_rhs_(s, U, R, nullptr);
        if (!strcmp(entry, "solve")) st = wcnst_solve_(s, U, INFINITY, 0.5, 3, nullptr, nullptr);
        if (!strcmp(entry, "noalloc"))
            st = wcnst_solve_noalloc_(&d, nullptr, U, INFINITY, 0.5, 3, nullptr, nullptr);
        printf("%d%s", st, k <= launches ? " " : "\n");
        last = hipSuccess;
        wcnst_destroy_(s);
        if (k > launches) return 0;
    }
}
