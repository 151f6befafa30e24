/* The part of the HIP host API that the library's host code calls, without a GPU: memory is host memory, launches do
 * nothing, and every call leaves a line in a log.  Loaded with RTLD_GLOBAL in front of the library, so that the library's
 * calls come here; tests then look at what it allocates, clears, waits for and launches.  (Registration of the device
 * code still goes to the HIP runtime, which needs no GPU for it; the kernels' names come here.) */
#define _GNU_SOURCE
#include <stdarg.h>
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;
enum { SUCCESS = 0, OUT_OF_MEMORY = 2 };

static char log_text[1 << 20];
static size_t log_len;
static size_t malloc_limit = (size_t)-1;      /* larger requests fail */
static int capturing;

static void note(const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    const int n = vsnprintf(log_text + log_len, sizeof(log_text) - log_len, fmt, ap);
    va_end(ap);
    if (n > 0 && log_len + (size_t)n < sizeof(log_text)) log_len += (size_t)n;
}

/* Streams and events are numbers that are never used twice, so that a use of one that is gone, a second destruction and one
 * left over can be told.  hipMalloc's blocks are counted. */
enum { STREAM = 1, EVENT = 2, MAX_HANDLES = 1 << 20 };
static unsigned char kind_of[MAX_HANDLES];    /* 0: not made yet, or destroyed */
static long next_handle = 1, live[3], blocks, misuses;
static const char *failing = "";              /* the call that fails */
static int fails(const char *call)
{
    if (strcmp(call, failing)) return SUCCESS;
    failing = "";
    return 1;
}
static void *handle(int kind)
{
    if (next_handle >= MAX_HANDLES) abort();
    kind_of[next_handle] = (unsigned char)kind;
    ++live[kind];
    return (void *)((uintptr_t)next_handle++ << 4);
}
static int known(void *h, int kind)
{
    const uintptr_t n = (uintptr_t)h >> 4;
    if (h && n < MAX_HANDLES && kind_of[n] == kind) return 1;
    ++misuses;
    return 0;
}
static int destroyed(void *h, int kind)
{
    if (!known(h, kind)) return 1;
    kind_of[(uintptr_t)h >> 4] = 0;
    --live[kind];
    return SUCCESS;
}
/* the null stream, one of the library's, or one of the caller's (2^30 and more) */
static void on_stream(void *st)
{
    if (!st || (uintptr_t)st >= 1u << 30) return;
    known(st, STREAM);
}
long stub_live(int kind) { return kind ? live[kind] : blocks; }
long stub_misuses(void) { return misuses; }
void stub_fail(const char *call) { static char name[64]; strncpy(name, call, sizeof(name) - 1); failing = name; }

const char *stub_log(void) { return log_text; }
void stub_clear_log(void) { log_text[0] = 0; log_len = 0; }
void stub_malloc_limit(size_t n) { malloc_limit = n; }
void stub_capturing(int on) { capturing = on; }

int hipGetDevice(int *dev) { *dev = 0; return SUCCESS; }
int hipDeviceGetAttribute(int *v, int attr, int dev) { (void)attr; (void)dev; *v = 0; return SUCCESS; }     /* unknown: the defaults stay */
int hipMalloc(void **p, size_t n)
{
    *p = n <= malloc_limit ? malloc(n) : NULL;
    blocks += *p != NULL;
    note("hipMalloc %zu%s\n", n, *p ? "" : " failed");
    return *p ? SUCCESS : OUT_OF_MEMORY;
}
int hipFree(void *p) { note("hipFree\n"); blocks -= p != NULL; free(p); return fails("hipFree"); }
int hipMemset(void *p, int v, size_t n) { note("hipMemset %zu\n", n); memset(p, v, n); return SUCCESS; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *st) { (void)kind; (void)st; memcpy(d, s, n); return SUCCESS; }
int hipDeviceSynchronize(void) { note("hipDeviceSynchronize\n"); return SUCCESS; }
int hipStreamSynchronize(void *st) { note("hipStreamSynchronize %p\n", st); return SUCCESS; }
int hipStreamCreateWithFlags(void **st, unsigned f) { (void)f; *st = handle(STREAM); return SUCCESS; }
int hipStreamDestroy(void *st) { note("hipStreamDestroy\n"); return destroyed(st, STREAM) || fails("hipStreamDestroy"); }
int hipStreamIsCapturing(void *st, int *status) { (void)st; *status = capturing; return SUCCESS; }
int hipStreamWaitEvent(void *st, void *ev, unsigned f) { on_stream(st); known(ev, EVENT); (void)f; note("hipStreamWaitEvent %p\n", st); return SUCCESS; }
int hipEventCreate(void **ev) { *ev = handle(EVENT); return SUCCESS; }
int hipEventCreateWithFlags(void **ev, unsigned f) { (void)f; note("hipEventCreateWithFlags\n"); *ev = handle(EVENT); return SUCCESS; }
int hipEventDestroy(void *ev) { note("hipEventDestroy\n"); return destroyed(ev, EVENT) || fails("hipEventDestroy"); }
int hipEventRecord(void *ev, void *st) { known(ev, EVENT); on_stream(st); note("hipEventRecord %p\n", st); return SUCCESS; }
int hipEventSynchronize(void *ev) { known(ev, EVENT); return SUCCESS; }
int hipEventElapsedTime(float *ms, void *a, void *b) { known(a, EVENT); known(b, EVENT); *ms = 1.0f; return SUCCESS; }
int hipFuncSetAttribute(const void *f, int attr, int v) { (void)f; (void)attr; (void)v; return SUCCESS; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int block, size_t lds) { (void)f; (void)block; (void)lds; *n = 1; return SUCCESS; }
static int last_error, launches_until_one_fails = -1;
void stub_fail_launch(int n) { launches_until_one_fails = n; }       /* after n that do not */
int hipGetLastError(void) { const int e = last_error; last_error = SUCCESS; return e; }
const char *hipGetErrorString(int e) { return e == OUT_OF_MEMORY ? "out of memory" : "error"; }

static struct { dim3_t grid, block; size_t lds; void *st; } pending;
int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t lds, void *st)
{
    pending.grid = grid; pending.block = block; pending.lds = lds; pending.st = st;
    return SUCCESS;
}
int __hipPopCallConfiguration(dim3_t *grid, dim3_t *block, size_t *lds, void **st)
{
    *grid = pending.grid; *block = pending.block; *lds = pending.lds; *st = pending.st;
    return SUCCESS;
}
static struct { const void *f; const char *name; } kernels[8192];
static int nkernels;
void __hipRegisterFunction(void **m, const void *f, char *df, const char *name, unsigned threads, void *tid, void *bid, void *bd, void *gd, int *ws)
{
    (void)m; (void)df; (void)threads; (void)tid; (void)bid; (void)bd; (void)gd; (void)ws;
    if (nkernels == sizeof kernels / sizeof *kernels) abort();
    kernels[nkernels].f = f;
    kernels[nkernels++].name = name;
}
static const char *name_of(const void *f)
{
    for (int i = 0; i < nkernels; ++i)
        if (kernels[i].f == f) return kernels[i].name;
    return "?";
}
int hipLaunchKernel(const void *f, dim3_t grid, dim3_t block, void **args, size_t lds, void *st)
{
    (void)args; (void)lds;
    on_stream(st);
    if (launches_until_one_fails >= 0 && launches_until_one_fails-- == 0) return last_error = 719;
    note("hipLaunchKernel %llu %llu %p %s\n", (unsigned long long)grid.x * grid.y * grid.z, (unsigned long long)block.x * block.y * block.z, st, name_of(f));
    return SUCCESS;
}
