/* A stand-in for the HIP runtime calls libbtrt.so makes, for tests of its host code without a GPU: device
 * memory is host memory, copies happen at once, kernels do nothing and take a millisecond each of the time events tell. A test
 * can make a copy fail and ask how many launches, of which threads, a stream got. */
#define __HIP_PLATFORM_AMD__ 1
#include <hip/hip_runtime_api.h>

#include <pthread.h>
#include <stdatomic.h>
#include <stdlib.h>
#include <string.h>

static atomic_int copies_left = -1; /* copies that still succeed; -1: all */
static atomic_int foreign;          /* launches on `watched` from other threads than the one that set it */
static atomic_int total;            /* launches on `watched` */
static hipStream_t watched;
static pthread_t owner;

void fake_fail_copy(int after) { atomic_store(&copies_left, after); }

void fake_watch(hipStream_t s)
{
    watched = s;
    owner = pthread_self();
    atomic_store(&foreign, 0);
    atomic_store(&total, 0);
}

int fake_foreign_launches(void) { return atomic_load(&foreign); }
int fake_launches(void) { return atomic_load(&total); }

hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int d) { (void)d; return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char* hipGetErrorString(hipError_t e) { (void)e; return "fake error"; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int d) { (void)a; (void)d; *v = 256; return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int d)
{
    (void)d;
    memset(p, 0, sizeof(*p));
    p->multiProcessorCount = 256;
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int block, size_t lds)
{
    (void)f; (void)block; (void)lds;
    *n = 2;
    return hipSuccess;
}

hipError_t hipMalloc(void** p, size_t n)
{
    *p = aligned_alloc(256, (n + 255) / 256 * 256);
    if (*p) memset(*p, 0, n);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void* p) { free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned f) { (void)f; return hipMalloc(p, n); }
hipError_t hipHostFree(void* p) { return hipFree(p); }
hipError_t hipGetSymbolAddress(void** p, const void* s) { (void)p; (void)s; return hipErrorInvalidSymbol; }

hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind k, hipStream_t s)
{
    (void)k; (void)s;
    const int left = atomic_load(&copies_left);
    if (left == 0) return hipErrorUnknown;
    if (left > 0) atomic_store(&copies_left, left - 1);
    memmove(dst, src, n);
    return hipSuccess;
}

static char handles[64];
static atomic_long launched; /* launches so far: the clock of events */
static long stamp[64];
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned f) { (void)f; *s = (hipStream_t)&handles[0]; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { (void)s; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { (void)s; return hipSuccess; }
static atomic_int events;
hipError_t hipEventCreate(hipEvent_t* e)
{
    *e = (hipEvent_t)&stamp[atomic_fetch_add(&events, 1) % 64];
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned f) { (void)f; return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { (void)e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s)
{
    (void)s;
    *(long*)e = atomic_load(&launched);
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) { (void)e; return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b)
{
    *ms = (float)(*(long*)b - *(long*)a); /* a millisecond a launch */
    return hipSuccess;
}

hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t lds, hipStream_t s)
{
    (void)f; (void)grid; (void)block; (void)args; (void)lds;
    atomic_fetch_add(&launched, 1);
    if (s == watched) {
        atomic_fetch_add(&total, 1);
        if (!pthread_equal(pthread_self(), owner)) atomic_fetch_add(&foreign, 1);
    }
    return hipSuccess;
}

/* The launch syntax <<<>>> passes its configuration through these. */
static __thread struct { dim3 grid, block; size_t lds; hipStream_t s; } conf;
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t s)
{
    conf.grid = grid;
    conf.block = block;
    conf.lds = lds;
    conf.s = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* s)
{
    *grid = conf.grid;
    *block = conf.block;
    *lds = conf.lds;
    *s = conf.s;
    return hipSuccess;
}
void** __hipRegisterFatBinary(const void* data) { (void)data; return (void**)handles; }
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterFunction(void** m, const void* f, char* d, const char* n, unsigned t, void* a, void* b, void* c, void* e,
                           int* w)
{
    (void)m; (void)f; (void)d; (void)n; (void)t; (void)a; (void)b; (void)c; (void)e; (void)w;
}
void __hipRegisterVar(void** m, void* v, char* d, char* n, int e, size_t z, int c, int g)
{
    (void)m; (void)v; (void)d; (void)n; (void)e; (void)z; (void)c; (void)g;
}
