/* A HIP runtime for host-logic tests without a GPU: device memory is host
 * memory, kernel launches do nothing, streams and events are numbers.  Every
 * call is counted by name; one call of a name can be made to fail; the order of
 * asynchronous copies and synchronisations is kept; event records can be held
 * until a number of threads has reached one.  Loaded before the library, whose
 * references to the HIP runtime then resolve to it. */
#include <pthread.h>
#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

enum { N_NAMES = 64, OK = 0, FAIL = 999 };
static pthread_mutex_t mu = PTHREAD_MUTEX_INITIALIZER;
static pthread_cond_t cv = PTHREAD_COND_INITIALIZER;
static const char *names[N_NAMES];
static int counts[N_NAMES], n_names;
static const char *fail_name;
static int fail_at, pending_copies;
static int gate_need, gate_seen;
static int n_alloc, watch, freed_watched;
static __thread int device, gate_passed;
static intptr_t next_handle = 0x1000;
static char symbol[2 * (1 << 19) * 8];

static int call(const char *name) {
    pthread_mutex_lock(&mu);
    int i = 0;
    while (i < n_names && strcmp(names[i], name)) ++i;
    if (i == n_names) names[n_names++] = name;
    const int k = ++counts[i];
    const int r = fail_name && !strcmp(fail_name, name) && k == fail_at ? FAIL : OK;
    pthread_mutex_unlock(&mu);
    return r;
}
static void *handle(void) { return (void *)__sync_add_and_fetch(&next_handle, 16); }

/* control, for the tests */
int fake_count(const char *name) {
    for (int i = 0; i < n_names; ++i)
        if (!strcmp(names[i], name)) return counts[i];
    return 0;
}
void fake_fail(const char *name, int after) {  /* the after-th call from now on fails; NULL: none */
    fail_name = name;
    fail_at = name ? fake_count(name) + after : 0;
}
int fake_pending_copies(void) { return pending_copies; }
void fake_watch(void) { watch = n_alloc; freed_watched = 0; }   /* from now on, count the frees */
int fake_freed_watched(void) { return freed_watched; }        /* of what is allocated by now */
void fake_device(int d) { device = d; }
void fake_gate(int threads) { gate_need = threads; gate_seen = 0; }

int hipGetDevice(int *d) { *d = device; return call("hipGetDevice"); }
/* allocations are numbered in a header of 64 bytes */
int hipMalloc(void **p, size_t n) {
    const int r = call("hipMalloc");
    *p = NULL;
    if (!r) {
        char *q = calloc(n + 64, 1);
        *(int *)q = __sync_add_and_fetch(&n_alloc, 1);
        *p = q + 64;
    }
    return r;
}
int hipFree(void *p) {
    if (p) {
        char *q = (char *)p - 64;
        if (*(int *)q <= watch) __sync_add_and_fetch(&freed_watched, 1);
        free(q);
    }
    return call("hipFree");
}
int hipMemcpy(void *d, const void *s, size_t n, int kind) {
    (void)kind;
    memcpy(d, s, n);
    return call("hipMemcpy");
}
int hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *st) {
    (void)kind; (void)st;
    memcpy(d, s, n);
    __sync_add_and_fetch(&pending_copies, 1);
    return call("hipMemcpyAsync");
}
int hipMemset(void *d, int v, size_t n) { memset(d, v, n); return call("hipMemset"); }
int hipMemsetAsync(void *d, int v, size_t n, void *st) { (void)st; memset(d, v, n); return call("hipMemsetAsync"); }
int hipDeviceSynchronize(void) { pending_copies = 0; return call("hipDeviceSynchronize"); }
int hipStreamSynchronize(void *s) { (void)s; pending_copies = 0; return call("hipStreamSynchronize"); }
int hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; *s = handle(); return call("hipStreamCreateWithFlags"); }
int hipStreamDestroy(void *s) { (void)s; return call("hipStreamDestroy"); }
int hipStreamWaitEvent(void *s, void *e, unsigned f) { (void)s; (void)e; (void)f; return call("hipStreamWaitEvent"); }
int hipStreamIsCapturing(void *s, int *st) { (void)s; *st = 0; return call("hipStreamIsCapturing"); }
int hipEventCreate(void **e) { *e = handle(); return call("hipEventCreate"); }
int hipEventCreateWithFlags(void **e, unsigned f) { (void)f; *e = handle(); return call("hipEventCreateWithFlags"); }
int hipEventDestroy(void *e) { (void)e; return call("hipEventDestroy"); }
int hipEventRecord(void *e, void *s) {
    (void)e; (void)s;
    if (gate_need && !gate_passed) {  /* each thread waits once, at its first record */
        gate_passed = 1;
        pthread_mutex_lock(&mu);
        if (++gate_seen == gate_need) pthread_cond_broadcast(&cv);
        while (gate_seen < gate_need) pthread_cond_wait(&cv, &mu);
        pthread_mutex_unlock(&mu);
    }
    return call("hipEventRecord");
}
int hipEventSynchronize(void *e) { (void)e; return call("hipEventSynchronize"); }
int hipEventElapsedTime(float *t, void *a, void *b) { (void)a; (void)b; *t = 1.0f; return call("hipEventElapsedTime"); }
int hipFuncSetAttribute(const void *f, int a, int v) { (void)f; (void)a; (void)v; return call("hipFuncSetAttribute"); }
int hipGetLastError(void) { return call("hipGetLastError"); }
const char *hipGetErrorString(int e) { return e ? "injected" : "none"; }
int hipGetSymbolAddress(void **p, const void *s) { (void)s; *p = symbol; return call("hipGetSymbolAddress"); }
typedef struct { uint32_t x, y, z; } dim3_;
static __thread struct { dim3_ g, b; size_t l; void *s; } config;
int __hipPushCallConfiguration(dim3_ g, dim3_ b, size_t l, void *s) {
    config.g = g; config.b = b; config.l = l; config.s = s;
    return OK;
}
int __hipPopCallConfiguration(dim3_ *g, dim3_ *b, size_t *l, void **s) {
    *g = config.g; *b = config.b; *l = config.l; *s = config.s;
    return OK;
}
int hipLaunchKernel(const void *f, dim3_ g, dim3_ b, void **a, size_t l, void *s) {
    (void)f; (void)g; (void)b; (void)a; (void)l; (void)s;
    return call("hipLaunchKernel");
}
