/* A HIP runtime that runs nothing: device memory is host memory up to a
 * limit, kernels are counted and not run, and an error stays until it is
 * asked for, as the real runtime's does.  Loaded before the library it takes
 * the place of the functions the library calls, so that its host code
 * (buffers, plans, launches) can be tested without a device. */
#include <hip/hip_runtime_api.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>

#define MAX_BLOCKS 4096
static struct { void *p; size_t n; } g_block[MAX_BLOCKS];
static size_t g_used, g_limit = (size_t)-1, g_peak;
static hipError_t g_last;
static long long g_launches, g_instantiated;
static int g_windows = 1;
static char g_scratch[64u << 20] __attribute__((aligned(256)));

/* what the tests set and read */
void rt_limit(size_t bytes) { g_limit = bytes; }
size_t rt_used(void) { return g_used; }
size_t rt_peak(int reset) {
    const size_t p = g_peak;
    if (reset) g_peak = g_used;
    return p;
}
long long rt_launches(void) { return g_launches; }
long long rt_instantiated(void) { return g_instantiated; }
/* windows of the next synchronous searches, whose reports (16 bytes each: event
 * records, minus the finished windows, first bad window) say that all ended */
void rt_windows(int B) { g_windows = B; }
/* fills the stack below the caller's frame */
__attribute__((noinline)) void rt_scribble(int v) {
    volatile char a[1 << 16];
    for (size_t k = 0; k < sizeof a; ++k) a[k] = (char)v;
}
hipError_t rt_last(void) { return g_last; }

static hipError_t fail(hipError_t e) {
    g_last = e;
    return e;
}

hipError_t hipMalloc(void **p, size_t n) {
    *p = NULL;
    if (n > g_limit || g_used > g_limit - n) return fail(hipErrorOutOfMemory);
    for (int k = 0; k < MAX_BLOCKS; ++k)
        if (!g_block[k].p) {
            /* zero pages, taken when touched */
            void *q = mmap(NULL, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
            if (q == MAP_FAILED) return fail(hipErrorOutOfMemory);
            *p = g_block[k].p = q;
            g_block[k].n = n;
            g_used += n;
            if (g_used > g_peak) g_peak = g_used;
            return hipSuccess;
        }
    return fail(hipErrorOutOfMemory);
}
hipError_t hipFree(void *p) {
    for (int k = 0; p && k < MAX_BLOCKS; ++k)
        if (g_block[k].p == p) {
            g_used -= g_block[k].n;
            g_block[k].p = NULL;
            munmap(p, g_block[k].n);
            return hipSuccess;
        }
    return p ? fail(hipErrorInvalidValue) : hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned flags) {
    (void)flags;
    if (posix_memalign(p, 256, n)) return fail(hipErrorOutOfMemory);
    memset(*p, 0, n);
    for (size_t k = 0; k < 3 && 16 * (k + 1) <= n; ++k) {
        const int v[4] = {0, 0, -g_windows, g_windows};
        memcpy((char *)*p + 16 * k, v, 16);
    }
    return hipSuccess;
}
hipError_t hipHostFree(void *p) {
    free(p);
    return hipSuccess;
}
hipError_t hipGetLastError(void) {
    const hipError_t e = g_last;
    g_last = hipSuccess;
    return e;
}
const char *hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "error"; }

hipError_t hipGetDeviceCount(int *n) {
    *n = 1;
    return hipSuccess;
}
hipError_t hipSetDevice(int d) { return d == 0 ? hipSuccess : fail(hipErrorInvalidDevice); }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int d) {
    (void)d;
    memset(p, 0, sizeof *p);
    p->multiProcessorCount = 256;
    p->sharedMemPerBlock = 160 * 1024;
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void *f, hipFuncAttribute a, int v) {
    (void)f, (void)a, (void)v;
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int threads, size_t lds) {
    (void)f;
    const int by_lds = lds ? (int)(160 * 1024 / lds) : 32, by_threads = 2048 / threads;
    *n = by_lds < by_threads ? by_lds : by_threads;
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *s) {
    (void)s;
    *p = g_scratch;
    return hipSuccess;
}

hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind k) {
    (void)k;
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t st) {
    (void)st;
    return hipMemcpy(d, s, n, k);
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t st) {
    (void)st;
    memset(d, v, n);
    return hipSuccess;
}

hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **a, size_t lds, hipStream_t s) {
    (void)f, (void)g, (void)b, (void)a, (void)lds, (void)s;
    ++g_launches;
    return hipSuccess;
}
hipError_t hipExtLaunchKernel(const void *f, dim3 g, dim3 b, void **a, size_t lds, hipStream_t s, hipEvent_t t0,
                              hipEvent_t t1, int flags) {
    (void)t0, (void)t1, (void)flags;
    return hipLaunchKernel(f, g, b, a, lds, s);
}
static struct { dim3 g, b; size_t lds; hipStream_t s; } g_call;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s) {
    g_call.g = g, g_call.b = b, g_call.lds = lds, g_call.s = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, hipStream_t *s) {
    *g = g_call.g, *b = g_call.b, *lds = g_call.lds, *s = g_call.s;
    return hipSuccess;
}
static void *g_module;
void **__hipRegisterFatBinary(const void *d) {
    (void)d;
    return &g_module;
}
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterFunction(void **m, const void *f, char *n, const char *d, unsigned t, void *a, void *b, void *c,
                           void *e, int *w) {
    (void)m, (void)f, (void)n, (void)d, (void)t, (void)a, (void)b, (void)c, (void)e, (void)w;
}
void __hipRegisterVar(void **m, void *v, char *n, const char *d, int e, size_t s, int c, int g) {
    (void)m, (void)v, (void)n, (void)d, (void)e, (void)s, (void)c, (void)g;
}

static int g_handle;
hipError_t hipStreamCreate(hipStream_t *s) {
    *s = (hipStream_t)&g_handle;
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) { return s ? hipSuccess : hipErrorInvalidValue; }
hipError_t hipStreamSynchronize(hipStream_t s) { return s ? hipSuccess : hipErrorInvalidValue; }
hipError_t hipEventCreate(hipEvent_t *e) {
    *e = (hipEvent_t)&g_handle;
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) { return e ? hipSuccess : hipErrorInvalidValue; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { return e && s ? hipSuccess : hipErrorInvalidValue; }
hipError_t hipEventSynchronize(hipEvent_t e) { return e ? hipSuccess : hipErrorInvalidValue; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t a, hipEvent_t b) {
    *ms = 0.0f;
    return a && b ? hipSuccess : hipErrorInvalidValue;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode m) {
    (void)m;
    return s ? hipSuccess : hipErrorInvalidValue;
}
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t *g) {
    *g = (hipGraph_t)&g_handle;
    return s ? hipSuccess : hipErrorInvalidValue;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t g, hipGraphNode_t *n, char *log, size_t size) {
    (void)n, (void)log, (void)size;
    *x = (hipGraphExec_t)&g_handle;
    ++g_instantiated;
    return g ? hipSuccess : hipErrorInvalidValue;
}
hipError_t hipGraphDestroy(hipGraph_t g) { return g ? hipSuccess : hipErrorInvalidValue; }
hipError_t hipGraphExecDestroy(hipGraphExec_t g) { return g ? hipSuccess : hipErrorInvalidValue; }
hipError_t hipGraphLaunch(hipGraphExec_t g, hipStream_t s) { return g && s ? hipSuccess : hipErrorInvalidValue; }
