/* The HIP runtime calls of libad.so without a device: loaded into a process
 * ahead of libad.so (its symbols then bind here), it runs no kernel and writes
 * down every launch, event record and stream wait, so that CPU tests can look
 * at what a call enqueues, also at sizes that no test could hold in memory, and
 * at what it does when a launch fails (fake_fail_at).  Device pointers are
 * never read; copies to the host give zeros. */
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;
typedef int err_t;                 /* hipError_t: 0 is success */
enum { MAX_FUNCS = 4096, LOG_BYTES = 1 << 22 };

static struct { const void *host; const char *name; } funcs[MAX_FUNCS];
static int n_funcs;
static char logbuf[LOG_BYTES];
static size_t log_at;
static long launches, fail_at = -1;
static err_t last_error;
static intptr_t next_handle = 16;  /* streams and events count up from here */
static struct { dim3_t g, b; size_t sh; void *st; } config;

#define LOG(...) do { \
        if (log_at + 512 < LOG_BYTES) log_at += (size_t)snprintf(logbuf + log_at, 512, __VA_ARGS__); \
    } while (0)

void fake_reset(long fail) { log_at = 0; logbuf[0] = 0; launches = 0; fail_at = fail; last_error = 0; }
const char *fake_log(void) { return logbuf; }
int fake_pending_error(void) { return last_error; }

void **__hipRegisterFatBinary(const void *d) { static void *m; (void)d; return &m; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterVar(void **m, void *v, char *h, char *d, int e, size_t s, int c, int g)
{ (void)m; (void)v; (void)h; (void)d; (void)e; (void)s; (void)c; (void)g; }
void __hipRegisterFunction(void **m, const void *host, char *dev, const char *name, unsigned lim, void *t, void *b,
                           void *bd, void *gd, int *w)
{
    (void)m; (void)dev; (void)lim; (void)t; (void)b; (void)bd; (void)gd; (void)w;
    if (n_funcs < MAX_FUNCS) { funcs[n_funcs].host = host; funcs[n_funcs].name = name; ++n_funcs; }
}
err_t __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t sh, void *st)
{ config.g = g; config.b = b; config.sh = sh; config.st = st; return 0; }
err_t __hipPopCallConfiguration(dim3_t *g, dim3_t *b, size_t *sh, void **st)
{ *g = config.g; *b = config.b; *sh = config.sh; *st = config.st; return 0; }

err_t hipLaunchKernel(const void *f, dim3_t g, dim3_t b, void **args, size_t sh, void *st)
{
    const char *name = "?";
    (void)args; (void)sh;
    for (int i = 0; i < n_funcs; ++i) if (funcs[i].host == f) name = funcs[i].name;
    ++launches;
    if (launches == fail_at) { last_error = 719; LOG("failed %.200s\n", name); return last_error; }
    LOG("launch %ld %.200s %u %u %u %u %u %u\n", (long)(intptr_t)st, name, g.x, g.y, g.z, b.x, b.y, b.z);
    return 0;
}
err_t hipGetLastError(void) { err_t e = last_error; last_error = 0; return e; }
const char *hipGetErrorString(err_t e) { return e ? "injected" : "no error"; }
err_t hipGetDevice(int *d) { *d = 0; return 0; }
err_t hipDeviceGetAttribute(int *v, int attr, int dev) { (void)attr; (void)dev; *v = 256; return 0; }
err_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *v, const void *f, int b, size_t s)
{ (void)f; (void)b; (void)s; *v = 4; return 0; }
err_t hipEventCreateWithFlags(void **e, unsigned f) { (void)f; *e = (void *)next_handle++; return 0; }
err_t hipEventCreate(void **e) { return hipEventCreateWithFlags(e, 0); }
err_t hipEventDestroy(void *e) { (void)e; return 0; }
err_t hipEventSynchronize(void *e) { (void)e; return 0; }
err_t hipEventRecord(void *e, void *st) { LOG("record %ld %ld\n", (long)(intptr_t)st, (long)(intptr_t)e); return 0; }
err_t hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; *s = (void *)next_handle++; return 0; }
err_t hipStreamDestroy(void *s) { (void)s; return 0; }
err_t hipStreamSynchronize(void *s) { (void)s; return 0; }
err_t hipStreamIsCapturing(void *s, int *c) { (void)s; *c = 0; return 0; }
err_t hipStreamWaitEvent(void *s, void *e, unsigned f)
{ (void)f; LOG("wait %ld %ld\n", (long)(intptr_t)s, (long)(intptr_t)e); return 0; }
err_t hipMemcpyAsync(void *dst, const void *src, size_t n, int kind, void *st)
{ (void)src; (void)st; if (kind == 2) memset(dst, 0, n); return 0; }
err_t hipMemsetAsync(void *dst, int v, size_t n, void *st) { (void)dst; (void)v; (void)n; (void)st; return 0; }
err_t hipHostMalloc(void **p, size_t n, unsigned f) { (void)f; *p = calloc(1, n); return *p ? 0 : 2; }
err_t hipGetSymbolAddress(void **p, const void *sym) { (void)sym; *p = (void *)(intptr_t)0x700000000000; return 0; }
err_t hipHostFree(void *p) { free(p); return 0; }
err_t hipHostGetDevicePointer(void **d, void *h, unsigned f) { (void)f; *d = h; return 0; }
