/* A stand-in for the HIP runtime calls that libge's host side makes, for tests
 * that run its planning and enqueueing without a GPU: memory is host memory, a
 * launch does nothing, and events, waits and launches are written to a log with
 * the calling thread.  Loaded with RTLD_GLOBAL before libge.so. */
#define _GNU_SOURCE
#include <pthread.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <time.h>

typedef struct { unsigned x, y, z; } dim3;

static pthread_mutex_t mu = PTHREAD_MUTEX_INITIALIZER;
static pthread_cond_t cv = PTHREAD_COND_INITIALIZER;
static char text[1 << 20];
static size_t used;
static int units = 256, fail_at = -1, launches, pause_ms, nthreads;
static uintptr_t next_handle = 0x1000;
static __thread int me, last_error;
static __thread struct { dim3 grid, block; size_t shared; void *stream; } config;

void fake_reset(int units_, int fail_at_, int pause_ms_)
{
    used = 0;
    text[0] = 0;
    units = units_;
    fail_at = fail_at_;
    pause_ms = pause_ms_;
    launches = 0;
}
const char *fake_log(void) { return text; }

static int tid(void)
{
    if (!me) me = ++nthreads;
    return me;
}
/* one line: what, stream, event (0: none), thread, workgroups and their threads;
 * with `mu` held */
static void line(const char *what, const void *stream, const void *event, unsigned groups,
                 unsigned threads)
{
    if (used < sizeof text - 128)
        used += (size_t)sprintf(text + used, "%s %lu %lu %d %u %u\n", what,
                                (unsigned long)(uintptr_t)stream, (unsigned long)(uintptr_t)event,
                                tid(), groups, threads);
}
static void *handle(void)
{
    pthread_mutex_lock(&mu);
    void *h = (void *)(next_handle += 16);
    pthread_mutex_unlock(&mu);
    return h;
}

int hipEventRecord(void *event, void *stream)
{
    static const void *first;
    pthread_mutex_lock(&mu);
    line("record", stream, event, 0, 0);
    if (pause_ms) {
        /* the first record waits for another thread's record of the same event */
        if (!first) {
            first = event;
            struct timespec t;
            clock_gettime(CLOCK_REALTIME, &t);
            t.tv_nsec += pause_ms * 1000000L;
            t.tv_sec += t.tv_nsec / 1000000000L;
            t.tv_nsec %= 1000000000L;
            while (first && pthread_cond_timedwait(&cv, &mu, &t) == 0) { }
            first = event;
        } else if (first == event) {
            first = NULL;
            pthread_cond_broadcast(&cv);
        }
    }
    pthread_mutex_unlock(&mu);
    return 0;
}
int hipStreamWaitEvent(void *stream, void *event, unsigned flags)
{
    (void)flags;
    pthread_mutex_lock(&mu);
    line("wait", stream, event, 0, 0);
    pthread_mutex_unlock(&mu);
    return 0;
}
int hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t shared, void *stream)
{
    (void)f, (void)args, (void)shared;
    pthread_mutex_lock(&mu);
    const int failed = launches++ == fail_at;
    line(failed ? "failed" : "launch", stream, NULL, grid.x, block.x);
    pthread_mutex_unlock(&mu);
    return last_error = failed ? 719 : 0;
}
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, void *stream)
{
    config.grid = grid;
    config.block = block;
    config.shared = shared;
    config.stream = stream;
    return 0;
}
int __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shared, void **stream)
{
    *grid = config.grid;
    *block = config.block;
    *shared = config.shared;
    *stream = config.stream;
    return 0;
}
int hipGetLastError(void)
{
    const int e = last_error;
    last_error = 0;
    return e;
}
const char *hipGetErrorString(int e) { return e ? "failed on purpose" : "no error"; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int *v, int attribute, int d)
{
    (void)attribute, (void)d;
    *v = units;
    return units > 0 ? 0 : 100;
}
int hipGetDevicePropertiesR0600(void *p, int d) { (void)p, (void)d; return 100; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int b, size_t s)
{
    (void)f, (void)b, (void)s;
    *n = 1;
    return 0;
}
int hipMalloc(void **p, size_t n) { *p = malloc(n); return units > 0 && *p ? 0 : 2; }
int hipFree(void *p) { free(p); return 0; }
int hipHostMalloc(void **p, size_t n, unsigned f) { (void)f; *p = calloc(1, n); return 0; }
int hipHostFree(void *p) { free(p); return 0; }
int hipHostGetDevicePointer(void **d, void *h, unsigned f) { (void)f; *d = h; return 0; }
int hipMemcpy(void *d, const void *s, size_t n, int k) { (void)k; memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *stream)
{
    (void)d, (void)s, (void)n, (void)k;
    pthread_mutex_lock(&mu);
    line("copy", stream, NULL, 0, 0);
    pthread_mutex_unlock(&mu);
    return 0;
}
int hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; *s = handle(); return 0; }
int hipStreamDestroy(void *s) { (void)s; return 0; }
int hipStreamSynchronize(void *s) { (void)s; return 0; }
int hipDeviceSynchronize(void) { return 0; }
int hipEventCreateWithFlags(void **e, unsigned f) { (void)f; *e = handle(); return 0; }
int hipEventDestroy(void *e) { (void)e; return 0; }
