/* The part of the HIP host API that the library's host code calls, without a GPU: memory is host memory, launches do
 * nothing, and every call leaves a line in a log.  Loaded with RTLD_GLOBAL in front of the library, so that the library's
 * calls come here; tests then look at what it allocates, clears, waits for and launches.  (Registration of the device
 * code still goes to the HIP runtime, which needs no GPU for it.) */
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

const char *stub_log(void) { return log_text; }
void stub_clear_log(void) { log_text[0] = 0; log_len = 0; }
void stub_malloc_limit(size_t n) { malloc_limit = n; }
void stub_capturing(int on) { capturing = on; }

int hipGetDevice(int *dev) { *dev = 0; return SUCCESS; }
int hipDeviceGetAttribute(int *v, int attr, int dev) { (void)attr; (void)dev; *v = 0; return SUCCESS; }     /* unknown: the defaults stay */
int hipMalloc(void **p, size_t n)
{
    *p = n <= malloc_limit ? malloc(n) : NULL;
    note("hipMalloc %zu%s\n", n, *p ? "" : " failed");
    return *p ? SUCCESS : OUT_OF_MEMORY;
}
int hipFree(void *p) { note("hipFree\n"); free(p); return SUCCESS; }
int hipMemset(void *p, int v, size_t n) { note("hipMemset %zu\n", n); memset(p, v, n); return SUCCESS; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *st) { (void)kind; (void)st; memcpy(d, s, n); return SUCCESS; }
int hipDeviceSynchronize(void) { note("hipDeviceSynchronize\n"); return SUCCESS; }
int hipStreamSynchronize(void *st) { note("hipStreamSynchronize %p\n", st); return SUCCESS; }
int hipStreamCreateWithFlags(void **st, unsigned f) { (void)f; *st = malloc(1); return SUCCESS; }
int hipStreamDestroy(void *st) { free(st); return SUCCESS; }
int hipStreamIsCapturing(void *st, int *status) { (void)st; *status = capturing; return SUCCESS; }
int hipStreamWaitEvent(void *st, void *ev, unsigned f) { (void)ev; (void)f; note("hipStreamWaitEvent %p\n", st); return SUCCESS; }
int hipEventCreate(void **ev) { *ev = malloc(1); return SUCCESS; }
int hipEventCreateWithFlags(void **ev, unsigned f) { (void)f; note("hipEventCreateWithFlags\n"); *ev = malloc(1); return SUCCESS; }
int hipEventDestroy(void *ev) { free(ev); return SUCCESS; }
int hipEventRecord(void *ev, void *st) { (void)ev; note("hipEventRecord %p\n", st); return SUCCESS; }
int hipEventSynchronize(void *ev) { (void)ev; return SUCCESS; }
int hipEventElapsedTime(float *ms, void *a, void *b) { (void)a; (void)b; *ms = 1.0f; return SUCCESS; }
int hipFuncSetAttribute(const void *f, int attr, int v) { (void)f; (void)attr; (void)v; return SUCCESS; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int block, size_t lds) { (void)f; (void)block; (void)lds; *n = 1; return SUCCESS; }
int hipGetLastError(void) { return SUCCESS; }
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
int hipLaunchKernel(const void *f, dim3_t grid, dim3_t block, void **args, size_t lds, void *st)
{
    (void)f; (void)args; (void)lds;
    note("hipLaunchKernel %llu %llu %p\n", (unsigned long long)grid.x * grid.y * grid.z, (unsigned long long)block.x * block.y * block.z, st);
    return SUCCESS;
}
