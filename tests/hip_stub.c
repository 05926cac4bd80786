/* A stand-in for the HIP runtime, for tests of the library's host code on a
 * machine without a GPU: device memory is host memory, kernels do nothing,
 * and every call that matters to a test is written to a log.  Loaded before
 * the library with global symbols (hip_stub.py), it takes the runtime's place.
 *
 * It keeps the rules the tests are about: a device-wide wait while a stream is
 * being captured fails and spoils the capture; waiting for a capturing stream
 * fails; a kernel launch or an allocation fails when a test asks for it. */
#include <stdarg.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <pthread.h>

typedef int err_t;
typedef struct { uint32_t x, y, z; } dim3_t;
enum { OK = 0, EMEM = 2, ELAUNCH = 719, ECAPTURE = 900, ESPOILT = 901 };

static pthread_mutex_t mu = PTHREAD_MUTEX_INITIALIZER;
static char *log_buf;
static size_t log_len, log_cap;
static err_t last_error;

static void say(const char *fmt, ...)
{
    char line[512];
    va_list ap;
    va_start(ap, fmt);
    const int n = vsnprintf(line, sizeof line, fmt, ap);
    va_end(ap);
    pthread_mutex_lock(&mu);
    if (log_len + (size_t)n + 2 > log_cap) {
        log_cap = 2 * (log_len + (size_t)n + 2);
        log_buf = realloc(log_buf, log_cap);
    }
    memcpy(log_buf + log_len, line, (size_t)n);
    log_len += (size_t)n;
    log_buf[log_len++] = '\n';
    log_buf[log_len] = 0;
    pthread_mutex_unlock(&mu);
}

/* ---- what tests call ---- */
static char fail_kernel[128];
static long fail_mallocs_from = -1, quiet;
const char *stub_log(void) { return log_buf ? log_buf : ""; }
void stub_clear(void) { log_len = 0; if (log_buf) log_buf[0] = 0; }
void stub_quiet(int q) { quiet = q; }
/* the next launch of a kernel whose (mangled) name holds `part` fails */
void stub_fail_launch(const char *part) { snprintf(fail_kernel, sizeof fail_kernel, "%s", part); }
/* allocations of at least `bytes` fail (-1: none) */
void stub_fail_malloc(long bytes) { fail_mallocs_from = bytes; }

/* ---- streams and captures ---- */
enum { MAX_CAPTURES = 64 };
static struct { void *stream; int spoilt; } captures[MAX_CAPTURES];
static int ncaptures;
static int find(void *s)
{
    for (int k = 0; k < ncaptures; ++k)
        if (captures[k].stream == s)
            return k;
    return -1;
}
err_t hipStreamCreateWithFlags(void **s, unsigned flags) { (void)flags; *s = malloc(16); return OK; }
err_t hipStreamDestroy(void *s) { free(s); return OK; }
err_t hipStreamBeginCapture(void *s, int mode)
{
    (void)mode;
    pthread_mutex_lock(&mu);
    captures[ncaptures].stream = s;
    captures[ncaptures++].spoilt = 0;
    pthread_mutex_unlock(&mu);
    return OK;
}
err_t hipStreamEndCapture(void *s, void **graph)
{
    pthread_mutex_lock(&mu);
    const int k = find(s);
    const int spoilt = k >= 0 && captures[k].spoilt;
    if (k >= 0)
        captures[k] = captures[--ncaptures];
    pthread_mutex_unlock(&mu);
    *graph = spoilt ? NULL : malloc(16);
    return spoilt ? ESPOILT : OK;
}
err_t hipStreamIsCapturing(void *s, int *status)
{
    const int k = find(s);
    *status = k < 0 ? 0 : captures[k].spoilt ? 2 : 1;
    return OK;
}
err_t hipStreamSynchronize(void *s)
{
    if (find(s) >= 0) {
        captures[find(s)].spoilt = 1;
        return last_error = ECAPTURE;
    }
    if (!quiet) say("sync %p", s);
    return OK;
}
err_t hipDeviceSynchronize(void)
{
    if (!quiet) say("devsync");
    for (int k = 0; k < ncaptures; ++k)
        captures[k].spoilt = 1;
    return ncaptures ? (last_error = ECAPTURE) : OK;
}
err_t hipGraphInstantiate(void **e, void *g, void *n, char *b, size_t z) { (void)g; (void)n; (void)b; (void)z; *e = malloc(16); return OK; }
err_t hipGraphDestroy(void *g) { free(g); return OK; }
err_t hipGraphExecDestroy(void *g) { free(g); return OK; }
err_t hipGraphLaunch(void *g, void *s) { (void)g; if (!quiet) say("graph %p", s); return OK; }

/* ---- events ---- */
err_t hipEventCreate(void **e) { *e = malloc(16); return OK; }
err_t hipEventCreateWithFlags(void **e, unsigned f) { (void)f; *e = malloc(16); return OK; }
err_t hipEventDestroy(void *e) { free(e); return OK; }
err_t hipEventRecord(void *e, void *s) { (void)e; (void)s; return OK; }
err_t hipEventSynchronize(void *e) { (void)e; return OK; }
err_t hipEventElapsedTime(float *ms, void *a, void *b) { (void)a; (void)b; *ms = 1.f; return OK; }

/* ---- memory ---- */
err_t hipMalloc(void **p, size_t bytes)
{
    *p = NULL;
    if (fail_mallocs_from >= 0 && (long)bytes >= fail_mallocs_from) {
        if (!quiet) say("nomem %zu", bytes);
        return last_error = EMEM;
    }
    if (posix_memalign(p, 512, bytes))
        return last_error = EMEM;
    memset(*p, 0, bytes);
    if (!quiet) say("malloc %zu %p", bytes, *p);
    return OK;
}
err_t hipFree(void *p)
{
    if (!quiet) say("free %p", p);
    free(p);
    return OK;
}
err_t hipHostMalloc(void **p, size_t bytes, unsigned flags) { (void)flags; *p = calloc(1, bytes); return *p ? OK : EMEM; }
err_t hipHostFree(void *p) { free(p); return OK; }
err_t hipMemcpy(void *d, const void *s, size_t n, int k) { (void)k; memmove(d, s, n); return OK; }
err_t hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *q) { (void)k; (void)q; memmove(d, s, n); return OK; }
err_t hipMemcpy2DAsync(void *d, size_t dp, const void *s, size_t sp, size_t w, size_t h, int k, void *q)
{
    (void)k; (void)q;
    for (size_t r = 0; r < h; ++r)
        memmove((char *)d + r * dp, (const char *)s + r * sp, w);
    return OK;
}
err_t hipMemset(void *d, int v, size_t n) { memset(d, v, n); return OK; }
err_t hipMemsetAsync(void *d, int v, size_t n, void *q) { (void)q; memset(d, v, n); return OK; }

/* ---- device ---- */
err_t hipGetDevice(int *d) { *d = 0; return OK; }
err_t hipSetDevice(int d) { (void)d; return OK; }
err_t hipDeviceGetAttribute(int *v, int a, int d) { (void)a; (void)d; *v = 256; return OK; }
err_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int t, size_t l) { (void)f; (void)t; (void)l; *n = 2; return OK; }
const char *hipGetErrorString(err_t e) { return e == OK ? "no error" : e == EMEM ? "out of memory" : "stub error"; }
err_t hipGetLastError(void) { const err_t e = last_error; last_error = OK; return e; }
err_t hipGetSymbolAddress(void **p, const void *sym) { (void)sym; static char words[4096]; *p = words; return OK; }

/* ---- kernels ---- */
enum { MAX_KERNELS = 4096 };
static struct { const void *host; const char *name; } kernels[MAX_KERNELS];
static int nkernels;
static const char *name_of(const void *f)
{
    for (int k = 0; k < nkernels; ++k)
        if (kernels[k].host == f)
            return kernels[k].name;
    return "?";
}
void **__hipRegisterFatBinary(const void *data) { (void)data; static void *h; return &h; }
void __hipUnregisterFatBinary(void **h) { (void)h; }
void __hipRegisterFunction(void **h, const void *host, char *dev, const char *name, unsigned t, void *a, void *b, void *c, void *d, int *w)
{
    (void)h; (void)dev; (void)t; (void)a; (void)b; (void)c; (void)d; (void)w;
    if (nkernels < MAX_KERNELS) {
        kernels[nkernels].host = host;
        kernels[nkernels++].name = name;
    }
}
void __hipRegisterVar(void **h, void *v, char *hv, char *n, int e, size_t s, int c, int g) { (void)h; (void)v; (void)hv; (void)n; (void)e; (void)s; (void)c; (void)g; }
static __thread struct { dim3_t g, b; size_t lds; void *s; } cfg;
err_t __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t lds, void *s) { cfg.g = g; cfg.b = b; cfg.lds = lds; cfg.s = s; return OK; }
err_t __hipPopCallConfiguration(dim3_t *g, dim3_t *b, size_t *lds, void **s) { *g = cfg.g; *b = cfg.b; *lds = cfg.lds; *s = cfg.s; return OK; }
static err_t launch(const void *f, dim3_t g, dim3_t b, size_t lds, void *s)
{
    const char *name = name_of(f);
    if (fail_kernel[0] && strstr(name, fail_kernel)) {
        fail_kernel[0] = 0;
        return last_error = ELAUNCH;
    }
    if (!quiet) say("launch %s %u %u %u %zu %p", name, g.x * g.y * g.z, b.x, g.x, lds, s);
    return OK;
}
err_t hipLaunchKernel(const void *f, dim3_t g, dim3_t b, void **a, size_t lds, void *s) { (void)a; return launch(f, g, b, lds, s); }
err_t hipLaunchCooperativeKernel(const void *f, dim3_t g, dim3_t b, void **a, unsigned lds, void *s) { (void)a; return launch(f, g, b, lds, s); }
err_t hipExtLaunchKernel(const void *f, dim3_t g, dim3_t b, void **a, size_t lds, void *s, void *e0, void *e1, int fl) { (void)a; (void)e0; (void)e1; (void)fl; return launch(f, g, b, lds, s); }
err_t hipFuncSetAttribute(const void *f, int attr, int v)
{
    (void)attr;
    if (!quiet) say("attr %s %d", name_of(f), v);
    return OK;
}
