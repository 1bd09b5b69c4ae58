/* The HIP calls the library's host side makes, on the CPU and without a GPU:
 * memory is host memory, kernels do nothing, and every call that orders work
 * is written to a log. A kernel that publishes the device header to the host
 * publishes stub_words instead (the header's words, then the totals). Loaded
 * before libspgemm.so with its symbols global, so the library binds to these.
 */
#include <stdarg.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef int err_t;
typedef void *stream_t, *event_t;
typedef struct { uint32_t x, y, z; } dim3_t;
typedef struct { unsigned long long *dst; int32_t nwords; uint32_t seq; } pub_t;

uint32_t stub_words[4096];
void *stub_capturing;        /* stream under capture */
char stub_fail_call[64];     /* a call of this name on stub_fail_on fails ... */
void *stub_fail_on;
int stub_fail_code;          /* ... with this code */

static char *lg;
static size_t lg_n, lg_cap;
static void note(const char *f, ...) {
    char line[256];
    va_list ap;
    va_start(ap, f);
    int n = vsnprintf(line, sizeof line, f, ap);
    va_end(ap);
    if (lg_n + n + 2 > lg_cap) lg = realloc(lg, lg_cap = 2 * (lg_cap + n + 2));
    memcpy(lg + lg_n, line, n);
    lg[lg_n + n] = '\n';
    lg[lg_n += n + 1] = 0;
}
const char *stub_log(void) { return lg ? lg : ""; }
void stub_clear(void) { lg_n = 0; if (lg) lg[0] = 0; }
static err_t fails(const char *call, void *on) {
    return strcmp(call, stub_fail_call) == 0 && on == stub_fail_on ? stub_fail_code : 0;
}

/* ------------------------------------------------------------- kernels */
static struct { const void *fun; char name[160]; } kernels[1024];
static int nkernels;
void **__hipRegisterFatBinary(const void *d) { (void)d; return calloc(1, sizeof(void *)); }
void __hipUnregisterFatBinary(void **h) { free(h); }
void __hipRegisterFunction(void **m, const void *fun, char *dev, const char *name, unsigned tl,
                           void *tid, void *bid, void *bd, void *gd, int *ws) {
    (void)m; (void)dev; (void)tl; (void)tid; (void)bid; (void)bd; (void)gd; (void)ws;
    if (nkernels < 1024) {
        kernels[nkernels].fun = fun;
        snprintf(kernels[nkernels++].name, sizeof kernels[0].name, "%s", name);
    }
}
void __hipRegisterVar(void **m, void *var, char *h, char *d, int ext, size_t n, int c, int g) {
    (void)m; (void)var; (void)h; (void)d; (void)ext; (void)n; (void)c; (void)g;
}
static struct { dim3_t g, b; size_t lds; stream_t s; } cfg;
err_t __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t lds, stream_t s) {
    cfg.g = g; cfg.b = b; cfg.lds = lds; cfg.s = s;
    return 0;
}
err_t __hipPopCallConfiguration(dim3_t *g, dim3_t *b, size_t *lds, stream_t *s) {
    *g = cfg.g; *b = cfg.b; *lds = cfg.lds; *s = cfg.s;
    return 0;
}
err_t hipLaunchKernel(const void *fun, dim3_t g, dim3_t b, void **args, size_t lds, stream_t s) {
    (void)b;
    const char *name = "?";
    for (int i = 0; i < nkernels; ++i)
        if (kernels[i].fun == fun) name = kernels[i].name;
    note("launch %s stream %p blocks %u lds %zu", name, s, g.x, lds);
    /* the argument that says where the header goes */
    static const struct { const char *name; int arg; } pubs[] = {
        {"k_place", 1}, {"k_scan_small", 2}, {"k_scan_down", 4}, {"k_publish", 1}, {"k_bv_scan", 1}};
    for (unsigned i = 0; i < sizeof pubs / sizeof pubs[0]; ++i) {
        if (!strstr(name, pubs[i].name)) continue;
        const pub_t *p = args[pubs[i].arg];
        if (!p->dst) break;
        note("publish %d words", p->nwords);
        for (int w = 0; w < p->nwords; ++w)
            p->dst[w] = stub_words[w] | (unsigned long long)p->seq << 32;
    }
    return 0;
}

/* -------------------------------------------------------------- memory */
static err_t get(void **p, size_t n) { return (*p = calloc(1, n ? n : 1)) ? 0 : 2; }
err_t hipMalloc(void **p, size_t n) { return get(p, n); }
err_t hipFree(void *p) { free(p); return 0; }
err_t hipMallocAsync(void **p, size_t n, stream_t s) {
    note("alloc %zu stream %p", n, s);
    return get(p, n);
}
err_t hipFreeAsync(void *p, stream_t s) { (void)s; free(p); return 0; }
err_t hipHostMalloc(void **p, size_t n, unsigned f) { (void)f; note("hostalloc %zu", n); return get(p, n); }
err_t hipHostFree(void *p) { note("hostfree"); free(p); return 0; }
err_t hipHostGetDevicePointer(void **d, void *h, unsigned f) { (void)f; *d = h; return 0; }
err_t hipGetSymbolAddress(void **p, const void *s) { (void)s; *p = 0; return 1; }
err_t hipMemcpy(void *d, const void *s, size_t n, int k) { (void)k; memcpy(d, s, n); return 0; }
err_t hipMemcpyAsync(void *d, const void *src, size_t n, int k, stream_t s) {
    note("copy %zu kind %d stream %p", n, k, s);
    memcpy(d, src, n);
    return 0;
}
err_t hipMemsetAsync(void *d, int v, size_t n, stream_t s) {
    note("memset %zu stream %p", n, s);
    memset(d, v, n);
    return 0;
}

/* --------------------------------------------------- streams and events */
static uintptr_t handle = 0x100000;
err_t hipStreamCreateWithFlags(stream_t *s, unsigned f) { (void)f; *s = (void *)(handle += 16); return 0; }
err_t hipStreamDestroy(stream_t s) { (void)s; return 0; }
err_t hipEventCreateWithFlags(event_t *e, unsigned f) { (void)f; *e = (void *)(handle += 16); return 0; }
err_t hipEventDestroy(event_t e) { (void)e; return 0; }
err_t hipEventElapsedTime(float *ms, event_t a, event_t b) { (void)a; (void)b; *ms = 0; return 0; }
err_t hipEventRecord(event_t e, stream_t s) {
    const err_t x = fails("hipEventRecord", s);
    note("record %p stream %p%s", e, s, x ? " failed" : "");
    return x;
}
err_t hipEventSynchronize(event_t e) { note("await %p", e); return 0; }
err_t hipStreamWaitEvent(stream_t s, event_t e, unsigned f) {
    (void)f;
    note("wait stream %p event %p", s, e);
    return 0;
}
err_t hipStreamSynchronize(stream_t s) {
    const err_t x = fails("hipStreamSynchronize", s);
    note("sync stream %p%s", s, x ? " failed" : "");
    return x;
}
err_t hipDeviceSynchronize(void) { note("sync device"); return 0; }
err_t hipStreamQuery(stream_t s) { (void)s; return 0; }
err_t hipStreamIsCapturing(stream_t s, int *st) { *st = s && s == stub_capturing; return 0; }
err_t hipGetLastError(void) { return 0; }
err_t hipGetDevice(int *d) { *d = 0; return 0; }
err_t hipDeviceGetAttribute(int *v, int a, int d) { (void)a; (void)d; *v = 256; return 0; }
err_t hipGetDevicePropertiesR0600(void *p, int d) { (void)p; (void)d; return 1; }
