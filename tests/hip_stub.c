/* A stand-in for the HIP runtime: what libnested_poisson.so calls of it, on the
 * host.  Loaded with RTLD_GLOBAL before the library, it takes the runtime's
 * place, so that the library's host side (validation, allocation, the schedule of
 * launches) runs on a machine without a GPU.  Device memory is host memory; a
 * kernel launch is written to a log and does nothing, except k_publish, which hands
 * the reduction slots (zero here) to the host: at once, or (stub_defer) only when the
 * stream is synchronised or queried often enough.
 */
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { unsigned x, y, z; } dim3_;

enum { SUCCESS = 0, OUT_OF_MEMORY = 2, NOT_READY = 600 };
#define MAX_FN 4096
static const void* fn_ptr[MAX_FN];
static const char* fn_name[MAX_FN];
static int n_fn;

static char* log_buf;
static size_t log_len, log_cap;
static long limit = -1, used, n_query, n_sync, n_malloc, n_free;
static int device_flags, defer, n_kernels_sync;

/* ---- what the tests set and read */
void stub_limit(long bytes) { limit = bytes; }  /* device memory; < 0: none */
void stub_flags(int f) { device_flags = f; }
void stub_defer(int queries) { defer = queries; }
long stub_used(void) { return used; }
long stub_queries(void) { return n_query; }
long stub_syncs(void) { return n_sync; }
long stub_live(void) { return n_malloc - n_free; }
const char* stub_log(void) { return log_buf ? log_buf : ""; }
void stub_clear(void)
{
    log_len = 0;
    if (log_buf) log_buf[0] = 0;
    n_query = n_sync = 0;
}

/* ---- modules */
void** __hipRegisterFatBinary(const void* d) { static void* h; (void)d; return &h; }
void __hipUnregisterFatBinary(void** h) { (void)h; }
void __hipRegisterVar(void** h, void* v, char* a, char* b, int e, size_t s, int c, int g)
{
    (void)h, (void)v, (void)a, (void)b, (void)e, (void)s, (void)c, (void)g;
}
void __hipRegisterFunction(void** h, const void* f, char* device, const char* name, unsigned t, void* a, void* b, void* c,
                           void* d, int* w)
{
    (void)h, (void)device, (void)t, (void)a, (void)b, (void)c, (void)d, (void)w;
    if (n_fn < MAX_FN) {
        fn_ptr[n_fn] = f;
        fn_name[n_fn++] = name;
    }
}

/* ---- launches */
static __thread struct { dim3_ g, b; size_t s; void* st; } cfg;
int __hipPushCallConfiguration(dim3_ g, dim3_ b, size_t s, void* st)
{
    cfg.g = g, cfg.b = b, cfg.s = s, cfg.st = st;
    return SUCCESS;
}
int __hipPopCallConfiguration(dim3_* g, dim3_* b, size_t* s, void** st)
{
    *g = cfg.g, *b = cfg.b, *s = cfg.s, *st = cfg.st;
    return SUCCESS;
}

static struct { unsigned long long *bits, *host; int n; unsigned seq; } pending;

static void publish(void)
{
    for (int t = 0; t < pending.n; t++) {
        const unsigned long long v = pending.bits[t], s = (unsigned long long)pending.seq << 32;
        pending.bits[t] = 0;
        __atomic_store_n(pending.host + 2 * t, s | (v & 0xffffffffULL), __ATOMIC_RELEASE);
        __atomic_store_n(pending.host + 2 * t + 1, s | (v >> 32), __ATOMIC_RELEASE);
    }
    pending.n = 0;
}

int hipLaunchKernel(const void* f, dim3_ g, dim3_ b, void** args, size_t shmem, void* st)
{
    const char* name = "?";
    char line[1024];
    (void)st;
    for (int i = 0; i < n_fn; i++)
        if (fn_ptr[i] == f) name = fn_name[i];
    const int m = snprintf(line, sizeof line, "%s %u %u %u %u %zu\n", name, g.x, g.y, g.z, b.x, shmem);
    if (log_len + m + 1 > log_cap) log_buf = realloc(log_buf, log_cap = 2 * (log_cap + m + 1));
    memcpy(log_buf + log_len, line, m + 1);
    log_len += m;
    if (strstr(name, "k_publish")) {
        if (pending.n) publish();
        pending.bits = *(unsigned long long**)args[0];
        pending.n = *(int*)args[1];
        pending.host = *(unsigned long long**)args[2];
        pending.seq = *(unsigned*)args[3];
        n_kernels_sync = 0;
        if (!defer) publish();
    }
    return SUCCESS;
}

/* ---- memory: the size in front of a block */
int hipMalloc(void** p, size_t n)
{
    if (limit >= 0 && used + (long)n > limit) {
        *p = NULL;
        return OUT_OF_MEMORY;
    }
    char* q = calloc(1, n + 64);
    *(size_t*)q = n;
    used += (long)n;
    n_malloc++;
    *p = q + 64;
    return SUCCESS;
}
int hipFree(void* p)
{
    if (!p) return SUCCESS;
    used -= (long)*(size_t*)((char*)p - 64);
    n_free++;
    free((char*)p - 64);
    return SUCCESS;
}
int hipHostMalloc(void** p, size_t n, unsigned fl) { (void)fl; *p = calloc(1, n); return SUCCESS; }
int hipHostFree(void* p) { free(p); return SUCCESS; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int k, void* st) { (void)k, (void)st; memcpy(d, s, n); return SUCCESS; }
int hipMemsetAsync(void* d, int v, size_t n, void* st) { (void)st; memset(d, v, n); return SUCCESS; }
int hipGetSymbolAddress(void** p, const void* s) { (void)s; *p = NULL; return 1; }

/* ---- device, stream, the rest */
int hipGetDeviceCount(int* n) { *n = 1; return SUCCESS; }
int hipGetDevice(int* d) { *d = 0; return SUCCESS; }
int hipSetDevice(int d) { (void)d; return SUCCESS; }
int hipGetDeviceFlags(unsigned* f) { *f = (unsigned)device_flags; return SUCCESS; }
int hipGetLastError(void) { return SUCCESS; }
const char* hipGetErrorString(int e) { return e == OUT_OF_MEMORY ? "out of memory" : "error"; }
int hipDeviceSynchronize(void) { return SUCCESS; }
int hipStreamSynchronize(void* st)
{
    (void)st;
    n_sync++;
    if (pending.n) publish();
    return SUCCESS;
}
int hipStreamQuery(void* st)
{
    (void)st;
    n_query++;
    if (!pending.n) return SUCCESS;
    if (++n_kernels_sync < defer) return NOT_READY;
    publish();
    return SUCCESS;
}
/* (no stream for recording: the coarse levels are launched one by one) */
int hipStreamCreateWithFlags(void** s, unsigned f) { (void)f; *s = NULL; return 1; }
int hipStreamDestroy(void* s) { (void)s; return SUCCESS; }
int hipStreamBeginCapture(void* s, int m) { (void)s, (void)m; return 1; }
int hipStreamEndCapture(void* s, void** g) { (void)s; *g = NULL; return 1; }
int hipGraphInstantiate(void** e, void* g, void* n, void* l, size_t z) { (void)e, (void)g, (void)n, (void)l, (void)z; return 1; }
int hipGraphLaunch(void* e, void* s) { (void)e, (void)s; return 1; }
int hipGraphDestroy(void* g) { (void)g; return SUCCESS; }
int hipGraphExecDestroy(void* g) { (void)g; return SUCCESS; }
int hipEventCreate(void** e) { *e = malloc(1); return SUCCESS; }
int hipEventDestroy(void* e) { free(e); return SUCCESS; }
int hipEventRecord(void* e, void* s) { (void)e, (void)s; return SUCCESS; }
int hipEventElapsedTime(float* ms, void* a, void* b) { (void)a, (void)b; *ms = 0; return SUCCESS; }
