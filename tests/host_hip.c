/* A stand-in for the HIP runtime, for tests of the library's host logic on a
 * machine without a GPU: memory is host memory, copies happen at once, and a
 * kernel launch is only written down (the kernel's name, its grid and the first
 * words of its first two arguments).  Built with the runtime's soname and loaded
 * before the library, so that the library binds to it. */
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3;
enum { kOutOfMemory = 2, kMaxLaunches = 65536, kMaxKernels = 1024 };

static struct { const void *host; const char *name; } kernels[kMaxKernels];
static int nkernels;
static struct { const char *name; uint32_t gx, gy; uint64_t word; int32_t second; } log_[kMaxLaunches];
static int nlog;
static int fail_device, fail_pinned, capturing, ncopies;

/* the tests' side */
void host_clear(void) { nlog = ncopies = 0; }
int host_copies(void) { return ncopies; }
int host_launches(void) { return nlog; }
const char *host_kernel(int i) { return log_[i].name; }
uint64_t host_word(int i) { return log_[i].word; }
int host_second(int i) { return log_[i].second; }
uint32_t host_grid(int i, int axis) { return axis ? log_[i].gy : log_[i].gx; }
void host_fail(int device, int pinned) { fail_device = device; fail_pinned = pinned; }
void host_capturing(int on) { capturing = on; }

/* the runtime's */
static dim3 cfg_grid, cfg_block;
static size_t cfg_shmem;
static void *cfg_stream;
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t m, void *s) {
    cfg_grid = g; cfg_block = b; cfg_shmem = m; cfg_stream = s;
    return 0;
}
int __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *m, void **s) {
    *g = cfg_grid; *b = cfg_block; *m = cfg_shmem; *s = cfg_stream;
    return 0;
}
void **__hipRegisterFatBinary(const void *d) { static void *m; (void)d; return &m; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterFunction(void **m, const void *host, char *dev, const char *name, unsigned lim,
                           void *a, void *b, void *c, void *d, int *w) {
    (void)m; (void)dev; (void)lim; (void)a; (void)b; (void)c; (void)d; (void)w;
    if (nkernels < kMaxKernels) {
        kernels[nkernels].host = host;
        kernels[nkernels++].name = name;
    }
}
void __hipRegisterVar(void **m, void *v, char *h, char *n, int e, size_t s, int c, int g) {
    (void)m; (void)v; (void)h; (void)n; (void)e; (void)s; (void)c; (void)g;
}
int hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t m, void *s) {
    (void)b; (void)m; (void)s;
    if (nlog == kMaxLaunches) return 1;
    log_[nlog].name = "?";
    for (int i = 0; i < nkernels; ++i)
        if (kernels[i].host == f) log_[nlog].name = kernels[i].name;
    log_[nlog].gx = g.x;
    log_[nlog].gy = g.y;
    memcpy(&log_[nlog].word, args[0], 8);
    memcpy(&log_[nlog].second, args[1], 4);
    ++nlog;
    return 0;
}
int hipMalloc(void **p, size_t n) {
    *p = fail_device ? NULL : aligned_alloc(256, (n + 255) / 256 * 256);
    return *p ? 0 : kOutOfMemory;
}
int hipFree(void *p) { free(p); return 0; }
int hipHostMalloc(void **p, size_t n, unsigned f) {
    (void)f;
    *p = fail_pinned ? NULL : malloc(n);
    return *p ? 0 : kOutOfMemory;
}
int hipHostFree(void *p) { free(p); return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *st) {
    (void)k; (void)st;
    ++ncopies;
    memcpy(d, s, n);
    return 0;
}
int hipMemsetAsync(void *d, int v, size_t n, void *st) { (void)st; memset(d, v, n); return 0; }
static void *token(void) { static char t; return &t; }
int hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; *s = token(); return 0; }
int hipStreamDestroy(void *s) { (void)s; return 0; }
int hipStreamSynchronize(void *s) { (void)s; return 0; }
int hipStreamGetDevice(void *s, int *d) { (void)s; *d = 0; return 0; }
int hipStreamIsCapturing(void *s, int *c) { (void)s; *c = capturing; return 0; }
int hipStreamBeginCapture(void *s, int m) { (void)s; (void)m; return 0; }
int hipStreamEndCapture(void *s, void **g) { (void)s; *g = token(); return 0; }
int hipGraphInstantiate(void **e, void *g, void **n, char *l, size_t b) {
    (void)g; (void)n; (void)l; (void)b;
    *e = token();
    return 0;
}
int hipGraphDestroy(void *g) { (void)g; return 0; }
int hipGraphExecDestroy(void *g) { (void)g; return 0; }
int hipGraphLaunch(void *g, void *s) { (void)g; (void)s; return 0; }
int hipGraphUpload(void *g, void *s) { (void)g; (void)s; return 0; }
int hipEventCreateWithFlags(void **e, unsigned f) { (void)f; *e = token(); return 0; }
int hipEventDestroy(void *e) { (void)e; return 0; }
int hipEventRecord(void *e, void *s) { (void)e; (void)s; return 0; }
int hipEventSynchronize(void *e) { (void)e; return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipSetDevice(int d) { (void)d; return 0; }
int hipGetSymbolAddress(void **p, const void *s) { (void)s; *p = token(); return 0; }
const char *hipGetErrorString(int e) { return e == kOutOfMemory ? "out of memory" : "error"; }
int hipGetLastError(void) { return 0; }
