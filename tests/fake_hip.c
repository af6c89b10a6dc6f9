/* A HIP runtime without a device, preloaded in front of the real one: device
   memory is host memory, copies are memcpy, kernels do nothing but enter a log
   of names and grids.  For tests of what the library's host code launches and
   copies. */
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;
typedef int err_t;

#define LOG 65536
static const char *names[LOG];
static dim3_t grids[LOG];
static int nlog;
static struct { const void *fn; const char *name; } fns[1024];
static int nfns;
static char fail_on[128];      /* launches of such kernels leave an error */
static int fail_copy = -1;     /* asynchronous copies until one fails, -1: none */
static err_t last;
static int32_t *h2d4;          /* destination of the last 4-byte copy to the device */
static int pending;            /* asynchronous copies since the last wait */

void fake_clear(void) { nlog = 0; }
int fake_count(void) { return nlog; }
int fake_copies_pending(void) { return pending; }
const char *fake_name(int k) { return names[k]; }
uint32_t fake_grid(int k, int d) { return d ? grids[k].y : grids[k].x; }
void fake_fail(const char *sub) { snprintf(fail_on, sizeof fail_on, "%s", sub); }
void fake_fail_copy(int n) { fail_copy = n; }
int32_t *fake_h2d4(void) { return h2d4; }

void **__hipRegisterFatBinary(const void *d) { static void *h; (void)d; return &h; }
void __hipUnregisterFatBinary(void **h) { (void)h; }
void __hipRegisterVar(void **h, void *v, char *a, const char *b, int e, size_t s, int c, int g) {}
void __hipRegisterFunction(void **h, const void *fn, char *a, const char *name, unsigned t,
                           void *x, void *y, void *z, void *w, int *u) {
    if (nfns < 1024) { fns[nfns].fn = fn; fns[nfns++].name = strdup(name); }
}

static struct { dim3_t g, b; size_t sh; void *st; } conf;
err_t __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t sh, void *st) {
    conf.g = g; conf.b = b; conf.sh = sh; conf.st = st;
    return 0;
}
err_t __hipPopCallConfiguration(dim3_t *g, dim3_t *b, size_t *sh, void **st) {
    *g = conf.g; *b = conf.b; *sh = conf.sh; *st = conf.st;
    return 0;
}
err_t hipLaunchKernel(const void *fn, dim3_t g, dim3_t b, void **args, size_t sh, void *st) {
    const char *name = "?";
    for (int k = 0; k < nfns; k++) if (fns[k].fn == fn) name = fns[k].name;
    if (nlog < LOG) { names[nlog] = name; grids[nlog++] = g; }
    if (fail_on[0] && strstr(name, fail_on)) last = 719;
    return last;
}
err_t hipGetLastError(void) { err_t e = last; last = 0; return e; }
const char *hipGetErrorString(err_t e) { return e ? "fake error" : "no error"; }

err_t hipMalloc(void **p, size_t n) { *p = calloc(1, n + 64); return *p ? 0 : 2; }
err_t hipFree(void *p) { free(p); return 0; }
err_t hipHostMalloc(void **p, size_t n, unsigned f) { return hipMalloc(p, n); }
err_t hipHostFree(void *p) { free(p); return 0; }
err_t hipMemcpy(void *d, const void *s, size_t n, int kind) { memcpy(d, s, n); return 0; }
err_t hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *st) {
    if (fail_copy >= 0 && fail_copy-- == 0) return 719;
    if (n == 4 && kind == 1) h2d4 = d;
    memcpy(d, s, n);
    pending++;
    return 0;
}
err_t hipMemset(void *d, int v, size_t n) { memset(d, v, n); return 0; }
err_t hipMemsetAsync(void *d, int v, size_t n, void *st) { memset(d, v, n); return 0; }
err_t hipGetSymbolAddress(void **p, const void *s) { return hipMalloc(p, 1 << 20); }
err_t hipGetDevice(int *d) { *d = 0; return 0; }
err_t hipDeviceSynchronize(void) { return 0; }
err_t hipDeviceGetAttribute(int *v, int a, int d) { *v = 256; return 0; }
err_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int t, size_t s) {
    *n = 4;
    return 0;
}

static void *handle(void) { return malloc(8); }
err_t hipStreamCreateWithFlags(void **s, unsigned f) { *s = handle(); return 0; }
err_t hipStreamDestroy(void *s) { free(s); return 0; }
err_t hipStreamSynchronize(void *s) { pending = 0; return 0; }
err_t hipStreamWaitEvent(void *s, void *e, unsigned f) { return 0; }
err_t hipStreamBeginCapture(void *s, int m) { return 0; }
err_t hipStreamEndCapture(void *s, void **g) { *g = handle(); return 0; }
err_t hipEventCreate(void **e) { *e = handle(); return 0; }
err_t hipEventCreateWithFlags(void **e, unsigned f) { *e = handle(); return 0; }
err_t hipEventDestroy(void *e) { free(e); return 0; }
err_t hipEventRecord(void *e, void *s) { return 0; }
err_t hipEventSynchronize(void *e) { return 0; }
err_t hipEventElapsedTime(float *ms, void *a, void *b) { *ms = 1.0f; return 0; }
err_t hipGraphInstantiate(void **x, void *g, void **n, char *l, size_t s) { *x = handle(); return 0; }
err_t hipGraphDestroy(void *g) { free(g); return 0; }
err_t hipGraphExecDestroy(void *x) { free(x); return 0; }
err_t hipGraphLaunch(void *x, void *s) { return 0; }
