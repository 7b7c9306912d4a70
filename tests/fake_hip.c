/* The calls of the HIP runtime that the library makes, on the CPU: device memory is host memory, kernels do nothing,
 * and copies and events wait on their streams while fake_hold(1) is set, so that tests of the host code can
 * stop time, count calls, run out of memory and make a launch fail.  Loaded with RTLD_GLOBAL ahead of the library. */
#define _GNU_SOURCE
#include <pthread.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

enum { Success = 0, InvalidValue = 1, OutOfMemory = 2, NotReady = 600, LaunchFailure = 719 };
typedef struct { uint32_t x, y, z; } dim3;

static pthread_mutex_t mu = PTHREAD_MUTEX_INITIALIZER;
static pthread_cond_t cv = PTHREAD_COND_INITIALIZER;
static int held, fail_graph, last_error;
static long n_attr, n_wait, n_copy;
static size_t budget = (size_t)1 << 40, used;

/* pending copies, in the order of their streams; an event holds the number of the last copy it waits for */
typedef struct { void *stream; const char *src; char *dst; size_t n; long id; int done; } Copy;
static Copy copies[1 << 16];
static int ncopies;
static long next_id = 1;
typedef struct { void *stream; long id; } Event;
#define MAXMEM 4096
static struct { char *p; size_t n; int device; } mem[MAXMEM];
static int nmem;

static void drain(void *stream, long upto) {
    for (int i = 0; i < ncopies; ++i)
        if (!copies[i].done && copies[i].stream == stream && copies[i].id <= upto) {
            memcpy(copies[i].dst, copies[i].src, copies[i].n);
            copies[i].done = 1;
        }
}
static void wait_for(void *stream, long upto) {
    ++n_wait;
    while (held) pthread_cond_wait(&cv, &mu);
    drain(stream, upto);
}

/* ---- controls ---- */
void fake_hold(int on) {
    pthread_mutex_lock(&mu);
    held = on;
    pthread_cond_broadcast(&cv);
    pthread_mutex_unlock(&mu);
}
void fake_fail_graph(int on) { fail_graph = on; }
void fake_budget(size_t b) { budget = b; }
size_t fake_used(void) { return used; }
long fake_attr_calls(void) { return n_attr; }
long fake_waits(void) { return n_wait; }
long fake_copies(void) { return n_copy; }
void fake_pin(void *p, size_t n) {
    pthread_mutex_lock(&mu);
    mem[nmem].p = p, mem[nmem].n = n, mem[nmem++].device = 0;
    pthread_mutex_unlock(&mu);
}
/* copies under way that read from [p, p + n) */
int fake_pending(const char *p, size_t n) {
    int k = 0;
    pthread_mutex_lock(&mu);
    for (int i = 0; i < ncopies; ++i) k += !copies[i].done && copies[i].src < p + n && p < copies[i].src + copies[i].n;
    pthread_mutex_unlock(&mu);
    return k;
}

/* ---- memory ---- */
static int alloc(void **p, size_t n, int device) {
    int r = Success;
    pthread_mutex_lock(&mu);
    if (device && used + n > budget) r = last_error = OutOfMemory;
    else {
        *p = aligned_alloc(256, (n + 255) / 256 * 256);
        mem[nmem].p = *p, mem[nmem].n = n, mem[nmem++].device = device;
        if (device) used += n;
    }
    pthread_mutex_unlock(&mu);
    return r;
}
static int release(void *p) {
    pthread_mutex_lock(&mu);
    for (int i = 0; i < nmem; ++i)
        if (p && mem[i].p == p) {
            if (mem[i].device) used -= mem[i].n;
            mem[i] = mem[--nmem];
            break;
        }
    pthread_mutex_unlock(&mu);
    free(p);
    return Success;
}
int hipMalloc(void **p, size_t n) { return alloc(p, n, 1); }
int hipHostMalloc(void **p, size_t n, unsigned f) { return alloc(p, n, 0); }
int hipFree(void *p) { return release(p); }
int hipHostFree(void *p) { return release(p); }
int hipMemGetInfo(size_t *fr, size_t *total) { return *fr = used < budget ? budget - used : 0, *total = budget, Success; }
int hipMemcpy(void *d, const void *s, size_t n, int k) { return Success; }
int hipMemset(void *d, int v, size_t n) { return Success; }
int hipMemsetAsync(void *d, int v, size_t n, void *st) { return Success; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *st) {
    pthread_mutex_lock(&mu);
    ++n_copy;
    copies[ncopies++] = (Copy){st, s, d, n, next_id++, 0};
    if (!held) drain(st, next_id);
    pthread_mutex_unlock(&mu);
    return Success;
}
int hipMemcpyToSymbol(const void *s, const void *p, size_t n, size_t o, int k) { return Success; }
int hipGetSymbolAddress(void **p, const void *s) {
    static char there[256];
    return *p = there, Success;
}
int hipPointerGetAttributes(int *at, const char *p) { /* the attributes start with the memory's type */
    int r = InvalidValue;
    pthread_mutex_lock(&mu);
    ++n_attr;
    for (int i = 0; i < nmem; ++i)
        if (p >= mem[i].p && p < mem[i].p + mem[i].n) r = Success, *at = mem[i].device ? 2 : 1;
    if (r) last_error = r;
    pthread_mutex_unlock(&mu);
    return r;
}

/* ---- streams, events, graphs ---- */
int hipStreamCreate(void **s) { return *s = malloc(8), Success; }
int hipStreamDestroy(void *s) { return free(s), Success; }
int hipStreamSynchronize(void *s) {
    pthread_mutex_lock(&mu);
    wait_for(s, next_id);
    pthread_mutex_unlock(&mu);
    return Success;
}
int hipDeviceSynchronize(void) { return Success; }
int hipEventCreateWithFlags(void **e, unsigned f) { return *e = calloc(1, sizeof(Event)), Success; }
int hipEventCreate(void **e) { return hipEventCreateWithFlags(e, 0); }
int hipEventDestroy(void *e) { return free(e), Success; }
int hipEventRecord(void *e, void *s) {
    pthread_mutex_lock(&mu);
    *(Event *)e = (Event){s, next_id - 1};
    pthread_mutex_unlock(&mu);
    return Success;
}
int hipEventSynchronize(void *e) {
    pthread_mutex_lock(&mu);
    const Event v = *(Event *)e;
    wait_for(v.stream, v.id);
    pthread_mutex_unlock(&mu);
    return Success;
}
int hipEventQuery(void *e) {
    pthread_mutex_lock(&mu);
    const int r = held ? NotReady : Success;
    if (!held) drain(((Event *)e)->stream, ((Event *)e)->id);
    pthread_mutex_unlock(&mu);
    return r;
}
int hipEventElapsedTime(float *ms, void *a, void *b) { return *ms = 0, Success; }
int hipStreamBeginCapture(void *s, int mode) { return Success; }
int hipStreamEndCapture(void *s, void **g) { return *g = malloc(8), Success; }
int hipGraphInstantiate(void **x, void *g, void *n, char *b, size_t z) { return *x = malloc(8), Success; }
int hipGraphLaunch(void *x, void *s) { return fail_graph ? (last_error = LaunchFailure) : Success; }
int hipGraphExecDestroy(void *x) { return free(x), Success; }
int hipGraphDestroy(void *g) { return free(g), Success; }

/* ---- device and kernels ---- */
int hipGetDeviceCount(int *n) { return *n = 1, Success; }
int hipGetDevice(int *d) { return *d = 0, Success; }
int hipSetDevice(int d) { return Success; }
const char *hipGetErrorString(int e) { return e == OutOfMemory ? "out of memory" : "error"; }
int hipGetLastError(void) {
    const int e = last_error;
    return last_error = 0, e;
}
int hipFuncSetAttribute(const void *f, int a, int v) { return Success; }
int hipLaunchKernel(const void *f, dim3 g, dim3 b, void **a, size_t l, void *s) { return Success; }
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t l, void *s) { return Success; }
int __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *l, void **s) {
    *g = *b = (dim3){1, 1, 1}, *l = 0, *s = 0;
    return Success;
}
void **__hipRegisterFatBinary(const void *d) {
    static void *h;
    return &h;
}
void __hipUnregisterFatBinary(void **h) {}
void __hipRegisterFunction(void **m, const void *f, char *d, const char *n, unsigned t, void *a, void *b, void *c, void *e, int *w) {}
void __hipRegisterVar(void **m, void *v, char *h, char *d, int e, size_t n, int c, int g) {}
