/* A host-only stand-in for the HIP runtime calls that the library makes: device memory is
 * host memory, kernels do nothing (but results are copied), and every call is written to a log.  Tests load it
 * before the library to look at the order of the library's calls and at what it does when
 * memory runs out, without a GPU. */
#define _GNU_SOURCE
#include <pthread.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>
#include <sys/syscall.h>
#include <unistd.h>

typedef struct { uint32_t x, y, z; } dim3_t;
typedef struct {
    char op[24];
    char name[72];
    int64_t tid, stream, a, b, bytes, dev;
} rec;

enum { MAX = 1 << 16, KERNELS = 4096 };
static rec log_[MAX];
static int64_t n_;
static int64_t in_use_, limit_ = (int64_t)1 << 62;
static pthread_mutex_t mu_ = PTHREAD_MUTEX_INITIALIZER;
static const void *fn_[KERNELS];
static const char *fname_[KERNELS];
static int nfn_;

static __thread int dev_;  /* the thread's current device */

static void put(const char *op, const char *name, const void *stream, const void *a,
                const void *b, size_t bytes)
{
    pthread_mutex_lock(&mu_);
    if (n_ < MAX) {
        rec *r = &log_[n_++];
        memset(r, 0, sizeof *r);
        strncpy(r->op, op, sizeof r->op - 1);
        if (name)
            strncpy(r->name, name, sizeof r->name - 1);
        r->tid = syscall(SYS_gettid);
        r->stream = (int64_t)stream;
        r->a = (int64_t)a;
        r->b = (int64_t)b;
        r->bytes = (int64_t)bytes;
        r->dev = dev_;
    }
    pthread_mutex_unlock(&mu_);
}

/* what the tests call */
int64_t fake_count(void) { return n_; }
const rec *fake_record(int64_t i) { return &log_[i]; }
void fake_clear(void) { n_ = 0; }
int64_t fake_in_use(void) { return in_use_; }
void fake_limit(int64_t bytes) { limit_ = bytes; }

/* memory: device and pinned blocks count against the limit alike */
static int get(void **p, size_t n, const char *op)
{
    pthread_mutex_lock(&mu_);
    size_t *q = in_use_ + (int64_t)n <= limit_ ? malloc(n + 256) : NULL;
    if (q)
        in_use_ += (int64_t)n;
    pthread_mutex_unlock(&mu_);
    put(op, NULL, NULL, q, NULL, n);
    if (!q)
        return 2; /* hipErrorOutOfMemory */
    q[0] = n;
    *p = (char *)q + 256;
    return 0;
}
static int put_back(void *p, const char *op)
{
    if (p) {
        size_t *q = (size_t *)((char *)p - 256);
        pthread_mutex_lock(&mu_);
        in_use_ -= (int64_t)q[0];
        pthread_mutex_unlock(&mu_);
        put(op, NULL, NULL, p, NULL, q[0]);
        free(q);
    }
    return 0;
}
int hipMalloc(void **p, size_t n) { return get(p, n, "malloc"); }
int hipHostMalloc(void **p, size_t n, unsigned f) { (void)f; return get(p, n, "hostmalloc"); }
int hipFree(void *p) { return put_back(p, "free"); }
int hipHostFree(void *p) { return put_back(p, "hostfree"); }
int hipMemcpy(void *d, const void *s, size_t n, int k)
{
    put("memcpy", NULL, NULL, d, s, n);
    (void)k;
    memcpy(d, s, n);
    return 0;
}
int hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *st)
{
    put("memcpyasync", NULL, st, d, s, n);
    (void)k;
    memcpy(d, s, n);
    return 0;
}
int hipMemset(void *d, int v, size_t n)
{
    put("memset", NULL, NULL, d, NULL, n);
    memset(d, v, n);
    return 0;
}
int hipMemsetAsync(void *d, int v, size_t n, void *st)
{
    put("memsetasync", NULL, st, d, NULL, n);
    memset(d, v, n);
    return 0;
}

/* streams, events, devices */
static intptr_t next_ = 0x1000;
static void *fresh(void)
{
    return (void *)__atomic_add_fetch(&next_, 16, __ATOMIC_SEQ_CST);
}
int hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; *s = fresh(); return 0; }
int hipStreamDestroy(void *s) { (void)s; return 0; }
int hipStreamSynchronize(void *s) { put("streamsync", NULL, s, NULL, NULL, 0); return 0; }
int hipStreamWaitEvent(void *s, void *e, unsigned f)
{
    (void)f;
    put("waitevent", NULL, s, e, NULL, 0);
    return 0;
}
int hipEventCreate(void **e) { *e = fresh(); return 0; }
int hipEventCreateWithFlags(void **e, unsigned f) { (void)f; *e = fresh(); return 0; }
int hipEventDestroy(void *e) { (void)e; return 0; }
int hipEventRecord(void *e, void *s) { put("eventrecord", NULL, s, e, NULL, 0); return 0; }
int hipEventSynchronize(void *e) { put("eventsync", NULL, NULL, e, NULL, 0); return 0; }
int hipEventQuery(void *e) { (void)e; return 0; }
int hipEventElapsedTime(float *ms, void *a, void *b) { (void)a; (void)b; *ms = 1.f; return 0; }
int hipDeviceSynchronize(void) { put("devicesync", NULL, NULL, NULL, NULL, 0); return 0; }
int hipGetDevice(int *d) { *d = dev_; return 0; }
int hipSetDevice(int d) { dev_ = d; return 0; }
int hipGetLastError(void) { return 0; }
const char *hipGetErrorString(int e) { return e == 2 ? "out of memory" : "error"; }
int hipDeviceGetAttribute(int *v, int a, int d) { (void)a; (void)d; *v = 256; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int b, size_t l)
{
    (void)f; (void)b; (void)l;
    *n = 4;
    return 0;
}

/* kernels */
typedef struct { /* ToHost of results.hip */
    const char *src[10];
    uint32_t off[10], bytes[10];
    int32_t n;
    char *dst;
} to_host;
static __thread struct { dim3_t g, b; size_t l; void *s; } cfg_;
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t l, void *s)
{
    cfg_.g = g;
    cfg_.b = b;
    cfg_.l = l;
    cfg_.s = s;
    return 0;
}
int __hipPopCallConfiguration(dim3_t *g, dim3_t *b, size_t *l, void **s)
{
    *g = cfg_.g;
    *b = cfg_.b;
    *l = cfg_.l;
    *s = cfg_.s;
    return 0;
}
int hipLaunchKernel(const void *f, dim3_t g, dim3_t b, void **args, size_t l, void *s)
{
    (void)g; (void)b; (void)l;
    const char *name = "?";
    for (int i = 0; i < nfn_; ++i)
        if (fn_[i] == f)
            name = fname_[i];
    put("launch", name, s, f, NULL, 0);
    if (strstr(name, "k_to_host")) {  /* the copies to pinned memory are done */
        const to_host *h = args[0];
        for (int i = 0; i < h->n; ++i) {
            put("copyout", NULL, s, h->dst + h->off[i], h->src[i], h->bytes[i]);
            memcpy(h->dst + h->off[i], h->src[i], h->bytes[i]);
        }
    }
    return 0;
}
static void *module_;
void **__hipRegisterFatBinary(const void *d) { (void)d; return &module_; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterFunction(void **m, const void *f, char *df, const char *name, unsigned t,
                           void *a, void *b, void *c, void *d, int *w)
{
    (void)m; (void)df; (void)t; (void)a; (void)b; (void)c; (void)d; (void)w;
    if (nfn_ < KERNELS) {
        fn_[nfn_] = f;
        fname_[nfn_++] = name;
    }
}
void __hipRegisterVar(void **m, void *v, char *hv, char *dv, int e, size_t s, int c, int g)
{
    (void)m; (void)v; (void)hv; (void)dv; (void)e; (void)s; (void)c; (void)g;
}
