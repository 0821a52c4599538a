/* A stand-in for the HIP runtime under the host code of libmipdhg.so: device
 * memory is host memory, kernels are only noted, and every call that matters
 * for ordering goes to a log ("what name-or-stream").  Loaded with global
 * symbols before the library, whose calls it then receives.  One call of one
 * name can be made to fail.  Streams and events are small numbers. */
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3;
typedef void *hipStream_t;
typedef int hipError_t;

static char *log_;
static size_t len_, cap_;
static char fail_[64];
static int skip_;
static uintptr_t next_ = 0x100;
static hipStream_t masked_ = (hipStream_t)-1;
static int last_err_;

static void note(const char *what, const char *name, hipStream_t s) {
    char line[512];
    int n = snprintf(line, sizeof(line), "%s %s %lx\n", what, name, (unsigned long)(uintptr_t)s);
    if (n > (int)sizeof(line) - 1) n = sizeof(line) - 1;
    if (len_ + n + 1 > cap_) log_ = realloc(log_, cap_ = 2 * (cap_ + n + 1));
    memcpy(log_ + len_, line, n + 1);
    len_ += n;
}
static hipError_t ret(const char *name) {
    if (!strcmp(fail_, name) && skip_-- == 0) {
        note("fail", name, 0);
        return last_err_ = 1;
    }
    return 0;
}
const char *shim_log(void) { return log_ ? log_ : ""; }
void shim_reset(void) { len_ = 0; last_err_ = 0; if (log_) log_[0] = 0; fail_[0] = 0; }
void shim_fail(const char *name, int skip) { snprintf(fail_, sizeof(fail_), "%s", name); skip_ = skip; }
void shim_mask(hipStream_t s) { masked_ = s; }

/* kernels, by the mangled name they are registered under */
static struct { const void *f; const char *name; } fn_[8192];
static int nfn_;
void **__hipRegisterFatBinary(const void *d) { static void *h; (void)d; return &h; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterVar(void **m, void *v, char *h, char *d, int e, size_t s, int c, int g) {
    (void)m; (void)v; (void)h; (void)d; (void)e; (void)s; (void)c; (void)g;
}
void __hipRegisterFunction(void **m, const void *f, char *d, const char *name, unsigned l, void *a, void *b, void *c,
                           void *e, int *w) {
    (void)m; (void)d; (void)l; (void)a; (void)b; (void)c; (void)e; (void)w;
    if (nfn_ < 8192) { fn_[nfn_].f = f; fn_[nfn_++].name = name; }
}
static dim3 g_, b_;
static size_t sh_;
static hipStream_t s_;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t sh, hipStream_t s) { g_ = g; b_ = b; sh_ = sh; s_ = s; return 0; }
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *sh, hipStream_t *s) { *g = g_; *b = b_; *sh = sh_; *s = s_; return 0; }
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t sh, hipStream_t s) {
    (void)args; (void)sh; (void)g; (void)b;
    const char *name = "?";
    for (int i = 0; i < nfn_; ++i)
        if (fn_[i].f == f) name = fn_[i].name;
    note("kernel", name, s);
    return ret("hipLaunchKernel");
}

hipError_t hipGetLastError(void) { int e = last_err_; last_err_ = 0; return e; }
const char *hipGetErrorString(hipError_t e) { return e ? "made to fail" : "no error"; }
hipError_t hipGetDevice(int *d) { *d = 0; return ret("hipGetDevice"); }
hipError_t hipDeviceGetAttribute(int *v, int a, int d) { (void)a; (void)d; *v = 256; return ret("hipDeviceGetAttribute"); }
hipError_t hipFuncSetAttribute(const void *f, int a, int v) { (void)f; (void)a; (void)v; return ret("hipFuncSetAttribute"); }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int b, size_t sh) {
    (void)f; (void)b; (void)sh; *n = 4; return ret("hipOccupancyMaxActiveBlocksPerMultiprocessor");
}
static hipError_t handle(const char *name, hipStream_t *h) { *h = (hipStream_t)next_++; return ret(name); }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned f) { (void)f; hipError_t e = handle("hipStreamCreateWithFlags", s); note("stream", "create", *s); return e; }
hipError_t hipStreamDestroy(hipStream_t s) { note("stream", "destroy", s); return 0; }
hipError_t hipStreamSynchronize(hipStream_t s) { note("sync", "stream", s); return ret("hipStreamSynchronize"); }
hipError_t hipStreamWaitEvent(hipStream_t s, void *e, unsigned f) { (void)e; (void)f; note("wait", "event", s); return ret("hipStreamWaitEvent"); }
hipError_t hipStreamBeginCapture(hipStream_t s, int m) { (void)m; note("capture", "begin", s); return ret("hipStreamBeginCapture"); }
hipError_t hipStreamEndCapture(hipStream_t s, void **g) { *g = (void *)next_++; note("capture", "end", s); return ret("hipStreamEndCapture"); }
hipError_t hipExtStreamGetCUMask(hipStream_t s, uint32_t n, uint32_t *m) {
    for (uint32_t i = 0; i < n; ++i) m[i] = s == masked_ ? 0xffu : 0xffffffffu;
    return ret("hipExtStreamGetCUMask");
}
hipError_t hipEventCreate(void **e) { *e = (void *)next_++; return ret("hipEventCreate"); }
hipError_t hipEventCreateWithFlags(void **e, unsigned f) { (void)f; *e = (void *)next_++; return ret("hipEventCreateWithFlags"); }
hipError_t hipEventDestroy(void *e) { (void)e; return 0; }
hipError_t hipEventRecord(void *e, hipStream_t s) { (void)e; (void)s; return ret("hipEventRecord"); }
hipError_t hipEventSynchronize(void *e) { (void)e; return ret("hipEventSynchronize"); }
hipError_t hipEventElapsedTime(float *ms, void *a, void *b) { (void)a; (void)b; *ms = 1.0f; return ret("hipEventElapsedTime"); }
hipError_t hipGraphInstantiate(void **x, void *g, void **n, char *l, size_t s) {
    (void)g; (void)n; (void)l; (void)s; *x = (void *)next_++; return ret("hipGraphInstantiate");
}
hipError_t hipGraphLaunch(void *x, hipStream_t s) { (void)x; note("graph", "launch", s); return ret("hipGraphLaunch"); }
hipError_t hipGraphDestroy(void *g) { (void)g; return 0; }
hipError_t hipGraphExecDestroy(void *x) { (void)x; return 0; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned f) { (void)f; *p = calloc(1, n); return ret("hipHostMalloc"); }
hipError_t hipHostFree(void *p) { free(p); return 0; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, int k) { (void)k; memmove(d, s, n); return ret("hipMemcpy"); }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, int k, hipStream_t st) { (void)k; (void)st; memmove(d, s, n); return ret("hipMemcpyAsync"); }
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t s) { (void)s; memset(d, v, n); return ret("hipMemsetAsync"); }
