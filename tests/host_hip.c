/* A HIP runtime without a device, preloaded by tests of the library's host code: device memory is only counted, kernels are
 * only written down (device name, grid and workgroup size, one line each), copies and waits do nothing.
 *   HOST_HIP_LOG      file that takes the launches (of a graph: one line)
 *   HOST_HIP_BUDGET   bytes of device memory (default: no limit); an allocation past it fails with hipErrorOutOfMemory
 *   HOST_HIP_GRAPHS   bytes that may be allocated for a graph to be instantiated (default: no limit)
 */
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <time.h>

typedef struct { unsigned x, y, z; } dim3;
enum { OK = 0, INVALID = 1, OOM = 2, NOT_READY = 600 };

static size_t used, peak, n_blocks;
static struct { void *p; size_t bytes; } blocks[1 << 16];
static struct { const void *f; const char *name; } kernels[1 << 12];
static int n_kernels;
static dim3 cfg_grid, cfg_block;
static size_t cfg_lds;
static void *cfg_stream;

static size_t limit(const char *name) { const char *v = getenv(name); return v ? strtoull(v, NULL, 10) : (size_t)-1; }

static double now(void) { struct timespec t; clock_gettime(CLOCK_MONOTONIC, &t); return t.tv_sec + 1e-9 * t.tv_nsec; }
static double busy_until;
/* streams and events are not done for so many seconds from now */
void host_hip_busy(double seconds) { busy_until = now() + seconds; }

size_t host_hip_peak(void) { return peak; }
size_t host_hip_used(void) { return used; }

int hipMalloc(void **p, size_t bytes) {
    if (used + bytes > limit("HOST_HIP_BUDGET") || n_blocks == sizeof blocks / sizeof *blocks) return OOM;
    used += bytes;
    if (used > peak) peak = used;
    *p = aligned_alloc(256, 256);
    blocks[n_blocks].p = *p; blocks[n_blocks++].bytes = bytes;
    return OK;
}
int hipFree(void *p) {
    for (size_t i = 0; i < n_blocks; ++i)
        if (blocks[i].p == p) { used -= blocks[i].bytes; blocks[i] = blocks[--n_blocks]; free(p); return OK; }
    return INVALID;
}
int hipHostMalloc(void **p, size_t bytes, unsigned flags) { (void)flags; *p = calloc(1, bytes); return *p ? OK : OOM; }
int hipHostFree(void *p) { free(p); return OK; }
int hipMemset(void *p, int v, size_t n) { (void)p; (void)v; (void)n; return OK; }
int hipMemsetAsync(void *p, int v, size_t n, void *s) { (void)p; (void)v; (void)n; (void)s; return OK; }
int hipMemcpy(void *d, const void *s, size_t n, int k) { (void)d; (void)s; (void)n; (void)k; return OK; }
/* the last upload (row table of a pass): its bytes, as many as fit */
static unsigned char uploaded[1 << 18];
static size_t n_uploaded;
size_t host_hip_uploaded(void *out, size_t cap) { memcpy(out, uploaded, cap < n_uploaded ? cap : n_uploaded); return n_uploaded; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *st) {
    (void)d; (void)st;
    if (k == 1 /* host to device */ && n <= sizeof uploaded) memcpy(uploaded, s, n_uploaded = n);
    return OK;
}
int hipGetDevice(int *d) { *d = 0; return OK; }
int hipDeviceGetAttribute(int *v, int a, int d) { (void)a; (void)d; *v = 256; return OK; }      /* compute units */
int hipDeviceSynchronize(void) { return OK; }
int hipGetLastError(void) { return OK; }
const char *hipGetErrorString(int e) { return e == OOM ? "out of memory" : "error"; }
int hipFuncSetAttribute(const void *f, int a, int v) { (void)f; (void)a; (void)v; return OK; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int b, size_t l) { (void)f; (void)b; (void)l; *n = 1; return OK; }
int hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; *s = malloc(1); return OK; }
int hipStreamDestroy(void *s) { free(s); return OK; }
int hipStreamSynchronize(void *s) { (void)s; return OK; }
int hipStreamQuery(void *s) { (void)s; return now() < busy_until ? NOT_READY : OK; }
int hipStreamWaitEvent(void *s, void *e, unsigned f) { (void)s; (void)e; (void)f; return OK; }
int hipEventCreate(void **e) { *e = malloc(1); return OK; }
int hipEventCreateWithFlags(void **e, unsigned f) { (void)f; return hipEventCreate(e); }
int hipEventDestroy(void *e) { free(e); return OK; }
int hipEventRecord(void *e, void *s) { (void)e; (void)s; return OK; }
int hipEventSynchronize(void *e) {
    (void)e;
    while (now() < busy_until) { struct timespec t = {0, 1000000}; nanosleep(&t, NULL); }
    return OK;
}
int hipStreamBeginCapture(void *s, int m) { (void)s; (void)m; return OK; }
int hipStreamEndCapture(void *s, void **g) { (void)s; *g = malloc(1); return OK; }
int hipGraphInstantiate(void **x, void *g, void *n, char *l, size_t b) {
    (void)g; (void)n; (void)l; (void)b;
    if (used > limit("HOST_HIP_GRAPHS")) return OOM;
    *x = malloc(1);
    return OK;
}
int hipGraphDestroy(void *g) { free(g); return OK; }
int hipGraphExecDestroy(void *x) { free(x); return OK; }
int hipGraphLaunch(void *x, void *s) {
    (void)x; (void)s;
    const char *log = getenv("HOST_HIP_LOG");
    FILE *o = log ? fopen(log, "a") : NULL;
    if (o) { fputs("graph 0 0 0 0\n", o); fclose(o); }
    return OK;
}

void **__hipRegisterFatBinary(const void *d) { (void)d; static void *h; return &h; }
void __hipUnregisterFatBinary(void **h) { (void)h; }
void __hipRegisterVar(void **m, void *v, char *h, char *d, int e, size_t n, int c, int g) { (void)m; (void)v; (void)h; (void)d; (void)e; (void)n; (void)c; (void)g; }
void __hipRegisterFunction(void **m, const void *f, char *d, const char *name, unsigned t, void *a, void *b, void *c, void *e, int *w) {
    (void)m; (void)d; (void)t; (void)a; (void)b; (void)c; (void)e; (void)w;
    if (n_kernels < (int)(sizeof kernels / sizeof *kernels)) { kernels[n_kernels].f = f; kernels[n_kernels++].name = name; }
}
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, void *s) { cfg_grid = g; cfg_block = b; cfg_lds = lds; cfg_stream = s; return OK; }
int __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, void **s) { *g = cfg_grid; *b = cfg_block; *lds = cfg_lds; *s = cfg_stream; return OK; }
int hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t lds, void *s) {
    (void)args; (void)lds; (void)s;
    const char *log = getenv("HOST_HIP_LOG");
    if (!log) return OK;
    FILE *o = fopen(log, "a");
    for (int i = 0; o && i < n_kernels; ++i)
        if (kernels[i].f == f) fprintf(o, "%s %u %u %u %u\n", kernels[i].name, g.x, g.y, g.z, b.x);
    if (o) fclose(o);
    return OK;
}
int hipLaunchCooperativeKernel(const void *f, dim3 g, dim3 b, void **args, unsigned lds, void *s) { return hipLaunchKernel(f, g, b, args, lds, s); }
