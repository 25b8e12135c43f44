/* A stand-in for the HIP runtime on machines without a GPU: allocations and copies in host
 * memory, kernel launches that do nothing, and allocations of one chosen size that fail.  The
 * tests of the library's host logic (buffers, error paths, launch choices) load it before
 * libnlte.so, whose runtime calls then end here. */
#define __HIP_PLATFORM_AMD__
#include <hip/hip_runtime_api.h>
#include <stdlib.h>
#include <string.h>

static size_t fail_size, live_bytes, sizes[1 << 16];
static size_t largest_var;
static int n_sizes, n_launches;
static hipError_t last = hipSuccess;

void fake_fail_size(size_t n) { fail_size = n; }
void fake_reset(void) { n_sizes = n_launches = 0; }
size_t fake_live(void) { return live_bytes; }
size_t fake_largest_var(void) { return largest_var; }
int fake_launches(void) { return n_launches; }
int fake_count(size_t n)
{
    int c = 0;
    for (int i = 0; i < n_sizes; ++i) c += sizes[i] == n;
    return c;
}

static hipError_t take(void **p, size_t n)
{
    *p = NULL;
    if (fail_size && n == fail_size) return last = hipErrorOutOfMemory;
    size_t *b = calloc(1, n + 64);
    if (!b) return last = hipErrorOutOfMemory;
    b[0] = n;
    *p = (char *)b + 64;
    live_bytes += n;
    if (n_sizes < (int)(sizeof sizes / sizeof *sizes)) sizes[n_sizes++] = n;
    return hipSuccess;
}
static hipError_t give(void *p)
{
    if (p) {
        size_t *b = (size_t *)((char *)p - 64);
        live_bytes -= b[0];
        free(b);
    }
    return hipSuccess;
}

hipError_t hipMalloc(void **p, size_t n) { return take(p, n); }
hipError_t hipFree(void *p) { return give(p); }
hipError_t hipHostMalloc(void **p, size_t n, unsigned f) { return (void)f, take(p, n); }
hipError_t hipHostFree(void *p) { return give(p); }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind k) { return (void)k, memmove(d, s, n), hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t t)
{
    return (void)k, (void)t, memmove(d, s, n), hipSuccess;
}
hipError_t hipMemcpyWithStream(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t t)
{
    return (void)k, (void)t, memmove(d, s, n), hipSuccess;
}
hipError_t hipMemset(void *d, int v, size_t n) { return memset(d, v, n), hipSuccess; }
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t t) { return (void)t, memset(d, v, n), hipSuccess; }
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **a, size_t l, hipStream_t t)
{
    (void)f, (void)g, (void)b, (void)a, (void)l, (void)t;
    ++n_launches;
    return hipSuccess;
}
hipError_t hipGetLastError(void)
{
    hipError_t e = last;
    last = hipSuccess;
    return e;
}
const char *hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "error"; }
hipError_t hipGetDeviceCount(int *n) { return *n = 1, hipSuccess; }
hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipSetDevice(int d) { return (void)d, hipSuccess; }
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int d) { return (void)a, (void)d, *v = 64, hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int d)
{
    (void)d;
    memset(p, 0, sizeof *p);
    p->multiProcessorCount = 256;
    p->warpSize = 64;
    strcpy(p->gcnArchName, "gfx950");
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *s) { return *p = (void *)s, hipSuccess; }
int hipGetStreamDeviceId(hipStream_t t) { return (void)t, 0; }
hipError_t hipStreamCreateWithFlags(hipStream_t *t, unsigned f) { return (void)f, *t = (hipStream_t)8, hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t t) { return (void)t, hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t t) { return (void)t, hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t t, hipEvent_t e, unsigned f) { return (void)t, (void)e, (void)f, hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { return *e = (hipEvent_t)8, hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { return (void)e, hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t t) { return (void)e, (void)t, hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t e) { return (void)e, hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t a, hipEvent_t b) { return (void)a, (void)b, *ms = 0.0f, hipSuccess; }

/* what the compiler emits at load time and around a launch */
static struct {
    dim3 g, b;
    size_t l;
    hipStream_t t;
} call;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t l, hipStream_t t)
{
    call.g = g, call.b = b, call.l = l, call.t = t;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *l, hipStream_t *t)
{
    *g = call.g, *b = call.b, *l = call.l, *t = call.t;
    return hipSuccess;
}
void **__hipRegisterFatBinary(const void *d) { return (void **)d; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterFunction(void **m, const void *h, char *d, const char *n, unsigned t, void *a, void *b, void *c, void *e, int *w)
{
    (void)m, (void)h, (void)d, (void)n, (void)t, (void)a, (void)b, (void)c, (void)e, (void)w;
}
void __hipRegisterVar(void **m, void *v, char *h, char *d, int e, size_t n, int c, int g)
{
    (void)m, (void)v, (void)h, (void)d, (void)e, (void)c, (void)g;
    if (n > largest_var) largest_var = n;
}
