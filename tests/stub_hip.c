/* A HIP runtime without a device, for tests of the library's host code on the CPU: memory is host memory, copies happen
 * at once, kernels are only logged by name (k_set_pred_next, which moves a slot's state, is carried out).  A test can cap
 * the memory and make a coming call fail.  Loaded with RTLD_GLOBAL before libwisv.so, whose HIP references then land here. */
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3;
enum { OK = 0, INVALID = 1, NO_MEMORY = 2, UNSUPPORTED = 801 };

static int last_error;
static int failed(int code) { return last_error = code; }

/* ---- what a test sets and reads */
static size_t limit = (size_t)-1, used;
static int fail_copy, fail_sync, fail_record, refuse_lds;   /* fail_*: the n-th coming call fails */
static char log_text[1 << 20];
static size_t log_len;
static void note(const char *what) {
    if (log_len + strlen(what) + 2 < sizeof log_text) log_len += sprintf(log_text + log_len, "%s\n", what);
}
void stub_limit(size_t bytes) { limit = bytes; }
size_t stub_used(void) { return used; }
void stub_fail(int copy, int sync, int record) { fail_copy = copy, fail_sync = sync, fail_record = record; }
void stub_refuse_lds(int on) { refuse_lds = on; }
const char *stub_log(void) { return log_text; }
void stub_log_clear(void) { log_len = 0, log_text[0] = 0; }
static int countdown(int *n) { return *n > 0 && --*n == 0; }

/* ---- memory: every block keeps its size in front */
static void *take(size_t n) {
    char *p = malloc(n + 64);
    if (!p) return 0;
    *(size_t *)p = n;
    return p + 64;
}
int hipMalloc(void **p, size_t n) {
    if (n > limit - used || !(*p = take(n))) return failed(NO_MEMORY);
    used += n;
    return OK;
}
int hipFree(void *p) {
    if (p) used -= *(size_t *)((char *)p - 64), free((char *)p - 64);
    return OK;
}
int hipHostMalloc(void **p, size_t n, unsigned flags) { return (void)flags, (*p = take(n)) ? OK : failed(NO_MEMORY); }
int hipHostFree(void *p) { return free((char *)p - 64), OK; }
int hipMemcpy(void *d, const void *s, size_t n, int kind) { return (void)kind, memcpy(d, s, n), OK; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *stream) {
    (void)stream, (void)kind;
    if (countdown(&fail_copy)) return failed(INVALID);
    note("copy");
    return memcpy(d, s, n), OK;
}
int hipMemcpy2DAsync(void *d, size_t dp, const void *s, size_t sp, size_t w, size_t h, int kind, void *stream) {
    (void)kind, (void)stream;
    for (size_t i = 0; i < h; ++i) memcpy((char *)d + i * dp, (const char *)s + i * sp, w);
    return OK;
}
int hipMemsetAsync(void *d, int v, size_t n, void *stream) { return (void)stream, memset(d, v, n), OK; }

/* ---- streams, events, graphs, devices */
int hipStreamCreate(void **s) { return *s = (void *)1, OK; }
int hipStreamDestroy(void *s) { return (void)s, OK; }
int hipStreamSynchronize(void *s) {
    (void)s;
    if (countdown(&fail_sync)) return failed(INVALID);
    return note("sync"), OK;
}
int hipEventCreate(void **e) { return *e = (void *)1, OK; }
int hipEventDestroy(void *e) { return (void)e, OK; }
int hipEventRecord(void *e, void *s) { return (void)e, (void)s, countdown(&fail_record) ? failed(INVALID) : OK; }
int hipEventSynchronize(void *e) { return (void)e, OK; }
int hipEventElapsedTime(float *ms, void *a, void *b) { return (void)a, (void)b, *ms = 0.f, OK; }
int hipStreamBeginCapture(void *s, int mode) { return (void)s, (void)mode, failed(UNSUPPORTED); }
int hipStreamEndCapture(void *s, void **g) { return (void)s, *g = 0, failed(UNSUPPORTED); }
int hipGraphInstantiate(void **x, void *g, void **n, char *b, size_t l) { return (void)g, (void)n, (void)b, (void)l, *x = 0, failed(UNSUPPORTED); }
int hipGraphLaunch(void *x, void *s) { return (void)x, (void)s, failed(UNSUPPORTED); }
int hipGraphDestroy(void *g) { return (void)g, OK; }
int hipGraphExecDestroy(void *x) { return (void)x, OK; }
int hipGetDeviceCount(int *n) { return *n = 1, OK; }
int hipSetDevice(int d) { return (void)d, OK; }
int hipGetLastError(void) {
    const int e = last_error;
    return last_error = OK, e;
}
const char *hipGetErrorString(int e) { return e == NO_MEMORY ? "out of memory" : e ? "injected failure" : "no error"; }
int hipFuncSetAttribute(const void *f, int attr, int v) { return (void)f, (void)attr, (void)v, refuse_lds ? failed(INVALID) : OK; }
int hipGetSymbolAddress(void **p, const void *sym) {
    (void)sym;
    static char place[64];
    return *p = place, OK;
}

/* ---- kernels */
static struct { const void *host; const char *name; } kernels[4096];
static int n_kernels;
void **__hipRegisterFatBinary(const void *data) { return (void)data, (void **)kernels; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterVar(void **m, void *v, char *h, char *d, int e, size_t n, int c, int g) { (void)m, (void)v, (void)h, (void)d, (void)e, (void)n, (void)c, (void)g; }
void __hipRegisterFunction(void **m, const void *host, char *dev, const char *name, unsigned threads, void *a, void *b, void *c, void *d, int *w) {
    (void)m, (void)dev, (void)threads, (void)a, (void)b, (void)c, (void)d, (void)w;
    if (n_kernels < 4096) kernels[n_kernels].host = host, kernels[n_kernels++].name = name;
}
static struct { dim3 grid, block; size_t lds; void *stream; } call;
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void *stream) {
    return call.grid = grid, call.block = block, call.lds = lds, call.stream = stream, OK;
}
int __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, void **stream) {
    return *grid = call.grid, *block = call.block, *lds = call.lds, *stream = call.stream, OK;
}
int hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t lds, void *stream) {
    (void)grid, (void)block, (void)lds, (void)stream;
    const char *name = "?";
    for (int i = 0; i < n_kernels; ++i)
        if (kernels[i].host == f) name = kernels[i].name;
    note(name);
    if (strstr(name, "k_set_pred_next")) {   /* (kv_len, pred_next, best, slot, row, new_len, parts) */
        int32_t *kv_len = *(int32_t **)args[0], *pred_next = *(int32_t **)args[1], *best = *(int32_t **)args[2];
        const int slot = *(int *)args[3], row = *(int *)args[4];
        if (row >= 0) pred_next[slot] = best[2 * 16 * row + 1];   /* the token of the row's first (value, token) pair */
        kv_len[slot] = *(int *)args[5];
    }
    return OK;
}
