/* A HIP runtime without a device, for tests of the library's host code on the CPU: it hands out
 * addresses, counts the bytes held, refuses what goes beyond a set capacity, and keeps a list of the kernels
 * launched.  Nothing is computed: copies to the host give zeros.  Loaded before the library under the
 * runtime's own soname, so that the library binds to it. */
#define _GNU_SOURCE
#include <pthread.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef int err_t;
enum { OK = 0, INVALID = 1, NO_MEMORY = 2 };
typedef struct { uint32_t x, y, z; } fake_dim3;

#define MAX_BLOCKS 4096
#define MAX_KERNELS 4096
static pthread_mutex_t mu = PTHREAD_MUTEX_INITIALIZER;
static struct { uintptr_t at; size_t bytes; } blocks[MAX_BLOCKS];
static struct { const void *host; char name[256]; } kernels[MAX_KERNELS];
static int nkernels, mallocs;
static uintptr_t next_at = (uintptr_t)1 << 40;
static size_t held, peak, capacity = (size_t)-1;
static err_t last;
static char *log_text;
static size_t log_used, log_cap;

/* ---- what the tests ask ---- */
void fake_capacity(size_t bytes) { capacity = bytes; }
size_t fake_held(void) { return held; }
size_t fake_peak(void) { return peak; }
int fake_mallocs(void) { return mallocs; }
/* launches since the last call, one "kernel blocks first_pointer_argument second" line each */
const char *fake_log(void)
{
    static char *out;
    free(out);
    out = strdup(log_text ? log_text : "");
    log_used = 0;
    if (log_text) log_text[0] = 0;
    return out;
}

static void note(const char *line)
{
    const size_t n = strlen(line);
    pthread_mutex_lock(&mu);
    if (log_used + n + 1 > log_cap) {
        log_cap = 2 * (log_used + n + 1);
        log_text = realloc(log_text, log_cap);
    }
    memcpy(log_text + log_used, line, n + 1);
    log_used += n;
    pthread_mutex_unlock(&mu);
}

/* ---- device memory ---- */
err_t hipMalloc(void **p, size_t bytes)
{
    err_t e = NO_MEMORY;
    pthread_mutex_lock(&mu);
    ++mallocs;
    for (int i = 0; i < MAX_BLOCKS && held + bytes <= capacity; ++i)
        if (!blocks[i].at) {
            blocks[i].at = next_at;
            blocks[i].bytes = bytes;
            *p = (void *)next_at;
            next_at += (bytes + 2 * 4096) / 4096 * 4096;
            held += bytes;
            if (held > peak) peak = held;
            e = OK;
            break;
        }
    pthread_mutex_unlock(&mu);
    return last = e;
}

err_t hipFree(void *p)
{
    err_t e = p ? INVALID : OK;
    pthread_mutex_lock(&mu);
    for (int i = 0; i < MAX_BLOCKS && p; ++i)
        if (blocks[i].at == (uintptr_t)p) {
            held -= blocks[i].bytes;
            blocks[i].at = 0;
            e = OK;
            break;
        }
    pthread_mutex_unlock(&mu);
    return e;
}

err_t hipHostMalloc(void **p, size_t bytes, unsigned flags)
{
    (void)flags;
    return (*p = calloc(1, bytes)) ? OK : NO_MEMORY;
}
err_t hipHostFree(void *p) { free(p); return OK; }

static void to_host(void *dst, size_t bytes, int kind) { if (kind == 2) memset(dst, 0, bytes); }
err_t hipMemcpy(void *dst, const void *src, size_t bytes, int kind) { (void)src; to_host(dst, bytes, kind); return OK; }
err_t hipMemcpyAsync(void *dst, const void *src, size_t bytes, int kind, void *st) { (void)src; (void)st; to_host(dst, bytes, kind); return OK; }
err_t hipMemsetAsync(void *dst, int v, size_t bytes, void *st)
{
    char line[128];
    (void)v; (void)st;
    snprintf(line, sizeof line, "memset %zu %p -\n", bytes, dst);
    note(line);
    return OK;
}

/* ---- kernels ---- */
void **__hipRegisterFatBinary(const void *data) { static void *h; (void)data; return &h; }
void __hipUnregisterFatBinary(void **h) { (void)h; }
void __hipRegisterVar(void **m, void *v, char *hv, char *name, int ext, size_t size, int c, int g)
{ (void)m; (void)v; (void)hv; (void)name; (void)ext; (void)size; (void)c; (void)g; }
void __hipRegisterFunction(void **m, const void *host, char *dev, const char *name, unsigned lim, void *a, void *b,
                           void *c, void *d, int *w)
{
    (void)m; (void)dev; (void)lim; (void)a; (void)b; (void)c; (void)d; (void)w;
    if (nkernels < MAX_KERNELS) {
        kernels[nkernels].host = host;
        snprintf(kernels[nkernels++].name, sizeof kernels[0].name, "%s", name);
    }
}
static __thread struct { fake_dim3 grid, block; size_t shared; void *stream; } config;
err_t __hipPushCallConfiguration(fake_dim3 grid, fake_dim3 block, size_t shared, void *stream)
{
    config.grid = grid; config.block = block; config.shared = shared; config.stream = stream;
    return OK;
}
err_t __hipPopCallConfiguration(fake_dim3 *grid, fake_dim3 *block, size_t *shared, void **stream)
{
    *grid = config.grid; *block = config.block; *shared = config.shared; *stream = config.stream;
    return OK;
}
err_t hipLaunchKernel(const void *host, fake_dim3 grid, fake_dim3 block, void **args, size_t shared, void *stream)
{
    const char *name = "?";
    char line[512];
    (void)block; (void)shared; (void)stream;
    for (int i = 0; i < nkernels; ++i)
        if (kernels[i].host == host) name = kernels[i].name;
    snprintf(line, sizeof line, "%s %u %p %p\n", name, grid.x, *(void **)args[0], *(void **)args[1]);
    note(line);
    return OK;
}
err_t hipGetSymbolAddress(void **p, const void *sym) { (void)sym; *p = (void *)0x1000; return OK; }

/* ---- the rest succeeds ---- */
err_t hipGetDevice(int *d) { *d = 0; return OK; }
err_t hipSetDevice(int d) { (void)d; return OK; }
err_t hipDeviceGetAttribute(int *v, int attr, int d) { (void)attr; (void)d; *v = 256; return OK; }
const char *hipGetErrorString(err_t e) { return e == NO_MEMORY ? "out of memory" : "error"; }
err_t hipGetLastError(void) { const err_t e = last; last = OK; return e; }
err_t hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; *s = (void *)0x10; return OK; }
err_t hipStreamDestroy(void *s) { (void)s; return OK; }
err_t hipStreamSynchronize(void *s) { (void)s; return OK; }
err_t hipEventCreateWithFlags(void **e, unsigned f) { (void)f; *e = (void *)0x20; return OK; }
err_t hipEventDestroy(void *e) { (void)e; return OK; }
err_t hipEventRecord(void *e, void *s) { (void)e; (void)s; return OK; }
err_t hipEventSynchronize(void *e) { (void)e; return OK; }
err_t hipStreamBeginCapture(void *s, int mode) { (void)s; (void)mode; return OK; }
err_t hipStreamEndCapture(void *s, void **g) { (void)s; *g = (void *)0x30; return OK; }
err_t hipGraphInstantiate(void **e, void *g, void *n, char *l, size_t sz) { (void)g; (void)n; (void)l; (void)sz; *e = (void *)0x40; return OK; }
err_t hipGraphLaunch(void *e, void *s) { (void)e; (void)s; return OK; }
err_t hipGraphExecDestroy(void *e) { (void)e; return OK; }
err_t hipGraphDestroy(void *g) { (void)g; return OK; }
