/* A stand-in for the HIP runtime without a device: memory is address ranges that nothing backs, copies
 * to the host give zeros, and every launch is reported to a callback instead of being run.  Loaded with
 * global visibility before the library, so that the library's calls end here. */
#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3;
typedef void (*launch_cb)(const char *name, uint32_t gx, uint32_t gy, uint32_t gz, uint32_t bx, uint32_t by,
                          uint32_t bz, size_t lds, void **args);
typedef void (*memory_cb)(int alloc, uint64_t addr, size_t bytes);

static launch_cb on_launch;
static memory_cb on_memory;
static long malloc_left = -1;   /* allocations until one fails, -1: none does */
static long malloc_fail;        /* allocations that fail before the others succeed */
static int launch_error;        /* what every launch returns to hipGetLastError */

void fake_set(launch_cb l, memory_cb m) { on_launch = l; on_memory = m; }
void fake_fail_malloc(long after) { malloc_left = after; }
void fake_fail_next(long n) { malloc_fail = n; }
void fake_fail_launches(int error) { launch_error = error; }

enum { MAX_KERNELS = 4096 };
static struct { const void *host; const char *name; } kernels[MAX_KERNELS];
static int n_kernels;
void **__hipRegisterFatBinary(const void *data) { (void)data; return (void **)kernels; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterFunction(void **m, const void *host, char *dev, const char *name, unsigned lim, void *a, void *b,
                           void *c, void *d, int *w) {
    (void)m; (void)dev; (void)lim; (void)a; (void)b; (void)c; (void)d; (void)w;
    if (n_kernels < MAX_KERNELS) { kernels[n_kernels].host = host; kernels[n_kernels++].name = name; }
}
void __hipRegisterVar(void **m, void *var, char *h, char *d, int e, size_t s, int c, int g) {
    (void)m; (void)var; (void)h; (void)d; (void)e; (void)s; (void)c; (void)g;
}

static struct { dim3 g, b; size_t lds; void *st; } cfg;
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, void *st) {
    cfg.g = g; cfg.b = b; cfg.lds = lds; cfg.st = st;
    return 0;
}
int __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, void **st) {
    *g = cfg.g; *b = cfg.b; *lds = cfg.lds; *st = cfg.st;
    return 0;
}
int hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t lds, void *st) {
    (void)st;
    if (launch_error) return launch_error;
    const char *name = "";
    for (int i = 0; i < n_kernels; ++i)
        if (kernels[i].host == f) name = kernels[i].name;
    if (on_launch) on_launch(name, g.x, g.y, g.z, b.x, b.y, b.z, lds, args);
    return 0;
}
int hipGetLastError(void) { return launch_error; }
const char *hipGetErrorString(int e) { (void)e; return "stand-in error"; }

static uint64_t next_addr = (uint64_t)1 << 44;
int hipMalloc(void **p, size_t n) {
    if (malloc_left == 0 || malloc_fail > 0) {   /* out of memory */
        if (malloc_fail > 0) --malloc_fail;
        return 2;
    }
    if (malloc_left > 0) --malloc_left;
    *p = (void *)next_addr;
    if (on_memory) on_memory(1, next_addr, n);
    next_addr += (n + 8191) & ~(uint64_t)4095;   /* a gap between ranges */
    return 0;
}
int hipFree(void *p) {
    if (p && on_memory) on_memory(0, (uint64_t)(uintptr_t)p, 0);
    return 0;
}
static int is_device(const void *p) { return (uint64_t)(uintptr_t)p >= ((uint64_t)1 << 44) && (uint64_t)(uintptr_t)p < next_addr; }
int hipMemcpy(void *d, const void *s, size_t n, int kind) {
    (void)s; (void)kind;
    if (!is_device(d)) memset(d, 0, n);
    return 0;
}
int hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *st) { (void)st; return hipMemcpy(d, s, n, kind); }
int hipMemset(void *d, int v, size_t n) { (void)d; (void)v; (void)n; return 0; }
int hipGetSymbolAddress(void **p, const void *s) { (void)s; return hipMalloc(p, 64 << 20); }
int hipSetDevice(int d) { (void)d; return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceSynchronize(void) { return 0; }
int hipDeviceGetAttribute(int *v, int attr, int dev) {
    (void)dev;
    *v = attr == 63 ? 256 : 160 * 1024;   /* hipDeviceAttributeMultiprocessorCount; else the LDS of a workgroup */
    return 0;
}
int hipFuncSetAttribute(const void *f, int a, int v) { (void)f; (void)a; (void)v; return 0; }
int hipStreamSynchronize(void *s) { (void)s; return 0; }
int hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; *s = (void *)8; return 0; }
int hipStreamDestroy(void *s) { (void)s; return 0; }
int hipStreamBeginCapture(void *s, int m) { (void)s; (void)m; return 0; }
int hipStreamEndCapture(void *s, void **g) { (void)s; *g = (void *)16; return 0; }
int hipGraphInstantiate(void **e, void *g, void *n, char *l, size_t s) { (void)g; (void)n; (void)l; (void)s; *e = (void *)24; return 0; }
int hipGraphLaunch(void *e, void *s) { (void)e; (void)s; return 0; }
int hipGraphDestroy(void *g) { (void)g; return 0; }
int hipGraphExecDestroy(void *g) { (void)g; return 0; }
int hipEventCreate(void **e) { *e = (void *)32; return 0; }
int hipEventDestroy(void *e) { (void)e; return 0; }
int hipEventRecord(void *e, void *s) { (void)e; (void)s; return 0; }
int hipEventSynchronize(void *e) { (void)e; return 0; }
int hipEventElapsedTime(float *ms, void *a, void *b) { (void)a; (void)b; *ms = 0.f; return 0; }
