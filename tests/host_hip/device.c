/* A HIP runtime without a device, loaded before the real one, for tests of the
 * library's host code on the CPU: allocations are numbers with a limit on their
 * sum, every copy and fill is checked against them, kernels do nothing, and
 * the clock can be moved on. */
#define _GNU_SOURCE
#include <pthread.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <sys/syscall.h>
#include <time.h>
#include <unistd.h>

enum { OK = 0, INVALID = 1, NO_MEMORY = 2, REFUSED = 900 };
enum { MAX_BLOCKS = 4096 };

static pthread_mutex_t mu = PTHREAD_MUTEX_INITIALIZER;
static struct { uint64_t p, n; } block[MAX_BLOCKS];
static int n_blocks;
static uint64_t next = 0x100000000000ull, used, limit = 288ull << 30, total = 288ull << 30;
static int last, refuse, capturing;
static long skip_s;

/* what a test sees and sets */
uint64_t dev_used(void) { return used; }
int dev_blocks(void) { return n_blocks; }
void dev_limit(uint64_t bytes) { limit = bytes; }
void dev_total(uint64_t bytes) { total = bytes; }
/* as while another thread captures: 1 the waits for the device, 2 allocation and release too */
void dev_refuse(int what) { refuse = what; }
/* the caller's stream records a graph: allocation is refused and ends the recording, as the runtime has it */
void dev_capture(int on) { capturing = on; }
int dev_capturing(void) { return capturing; }
void dev_skip(long seconds) { skip_s += seconds; }

/* the last copy to the device */
static unsigned char *upload;
static uint64_t n_upload;
uint64_t dev_upload(void *out, uint64_t cap)
{
    memcpy(out, upload, cap < n_upload ? cap : n_upload);
    return n_upload;
}

int clock_gettime(clockid_t id, struct timespec *t)
{
    const int rc = (int)syscall(SYS_clock_gettime, id, t);
    if (id == CLOCK_MONOTONIC) t->tv_sec += skip_s;
    return rc;
}

static int set(int e)
{
    if (e) last = e;
    return e;
}

static void wrong(const char *what, const void *p, uint64_t n)
{
    fprintf(stderr, "device: %s at %p, %llu bytes\n", what, p, (unsigned long long)n);
    abort();
}

int hipMalloc(void **p, size_t n)
{
    if (refuse > 1 || capturing) {
        capturing = 0;
        return set(REFUSED);
    }
    pthread_mutex_lock(&mu);
    if (used + n > limit || n_blocks == MAX_BLOCKS) {
        pthread_mutex_unlock(&mu);
        return set(NO_MEMORY);
    }
    block[n_blocks].p = next;
    block[n_blocks++].n = n;
    *p = (void *)next;
    next += (n + 0x1FFFFFull) & ~0xFFFFFull;
    used += n;
    pthread_mutex_unlock(&mu);
    return OK;
}

int hipFree(void *p)
{
    if (!p) return OK;
    if (refuse > 1) return set(REFUSED);
    pthread_mutex_lock(&mu);
    int i = 0;
    while (i < n_blocks && block[i].p != (uint64_t)p) ++i;
    if (i == n_blocks) wrong("free of what is not allocated", p, 0);
    used -= block[i].n;
    block[i] = block[--n_blocks];
    pthread_mutex_unlock(&mu);
    return OK;
}

int hipMallocAsync(void **p, size_t n, void *s) { (void)s; return hipMalloc(p, n); }
int hipFreeAsync(void *p, void *s) { (void)s; return hipFree(p); }

static int on_device(const void *p) { return (uint64_t)p >> 44 == 1; }

static void check(const void *p, uint64_t n)
{
    pthread_mutex_lock(&mu);
    for (int i = 0; i < n_blocks; ++i)
        if (block[i].p <= (uint64_t)p && (uint64_t)p + n <= block[i].p + block[i].n) {
            pthread_mutex_unlock(&mu);
            return;
        }
    wrong("copy or fill past an allocation", p, n);
}

int hipMemsetAsync(void *p, int v, size_t n, void *s)
{
    (void)v; (void)s;
    check(p, n);
    return OK;
}

int hipMemcpy(void *d, const void *q, size_t n, int kind)
{
    (void)kind;
    if (on_device(q)) check(q, n);
    if (on_device(d)) {
        check(d, n);
        if (!on_device(q) && n && (upload = realloc(upload, n))) memcpy(upload, q, n_upload = n);
    } else if (on_device(q)) memset(d, 0, n);
    else memcpy(d, q, n);
    return OK;
}
int hipMemcpyAsync(void *d, const void *q, size_t n, int kind, void *s) { (void)s; return hipMemcpy(d, q, n, kind); }

int hipMemGetInfo(size_t *f, size_t *t) { *f = total - used; *t = total; return OK; }
int hipHostMalloc(void **p, size_t n, unsigned f) { (void)f; *p = calloc(1, n ? n : 1); return *p ? OK : set(NO_MEMORY); }
int hipHostFree(void *p) { free(p); return OK; }
int hipHostGetDevicePointer(void **d, void *h, unsigned f) { (void)f; *d = h; return OK; }
int hipGetDevice(int *d) { *d = 0; return OK; }
int hipGetLastError(void) { const int e = last; last = 0; return e; }
int hipDeviceSynchronize(void) { return refuse ? set(REFUSED) : OK; }
int hipStreamSynchronize(void *s) { (void)s; return OK; }
int hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; *s = malloc(1); return OK; }
int hipStreamDestroy(void *s) { free(s); return OK; }
int hipStreamIsCapturing(void *s, int *on) { (void)s; *on = capturing; return OK; }
int hipStreamBeginCapture(void *s, int m) { (void)s; (void)m; return OK; }
int hipStreamEndCapture(void *s, void **g) { (void)s; *g = malloc(1); return OK; }
int hipGraphInstantiate(void **e, void *g, void *n, char *b, size_t l) { (void)g; (void)n; (void)b; (void)l; *e = malloc(1); return OK; }
int hipGraphDestroy(void *g) { free(g); return OK; }
int hipGraphExecDestroy(void *e) { free(e); return OK; }
int hipGraphLaunch(void *e, void *s) { (void)e; (void)s; return OK; }
int hipEventCreate(void **e) { *e = malloc(1); return OK; }
int hipEventDestroy(void *e) { free(e); return OK; }
int hipEventRecord(void *e, void *s) { (void)e; (void)s; return OK; }
int hipEventSynchronize(void *e) { (void)e; return OK; }
int hipEventElapsedTime(float *ms, void *a, void *b) { (void)a; (void)b; *ms = 0.01f; return OK; }

typedef struct { unsigned x, y, z; } dim3_t;
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t m, void *s) { (void)g; (void)b; (void)m; (void)s; return OK; }
int __hipPopCallConfiguration(dim3_t *g, dim3_t *b, size_t *m, void **s)
{
    const dim3_t one = {1, 1, 1};
    *g = *b = one;
    *m = 0;
    *s = 0;
    return OK;
}
int hipLaunchKernel(const void *f, dim3_t g, dim3_t b, void **a, size_t m, void *s)
{
    (void)f; (void)g; (void)b; (void)a; (void)m; (void)s;
    return OK;
}
