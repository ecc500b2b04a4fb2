/* Stands in for the HIP runtime on the CPU: device memory is host memory, a
 * kernel launch is recorded (name, workgroups) and not run, chosen launches can
 * be made to fail, and events report a made-up time that differs from call to
 * call.  Loaded with RTLD_GLOBAL ahead of the library, whose runtime calls then
 * resolve here. */
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;

enum { MAX_FUNCS = 1024, MAX_LOG = 1 << 16 };
static struct { const void *host; const char *name; } funcs[MAX_FUNCS];
static int n_funcs;
static struct { const char *name; uint32_t grid, threads; } log_[MAX_LOG];
static int n_log, last_error;
static char fail_name[256];
static int fail_times;
static uint32_t noise = 12345;

void rec_clear(void) { n_log = 0; }
int rec_count(void) { return n_log; }
const char *rec_name(int i) { return log_[i].name; }
int rec_grid(int i) { return (int)log_[i].grid; }
int rec_threads(int i) { return (int)log_[i].threads; }
void rec_fail(const char *name, int times) { strncpy(fail_name, name, sizeof fail_name - 1); fail_times = times; }

void **__hipRegisterFatBinary(const void *d) { (void)d; static void *h; return &h; }
void __hipUnregisterFatBinary(void **h) { (void)h; }
void __hipRegisterVar(void **h, void *v, char *hv, char *dv, int e, size_t s, int c, int g)
{
    (void)h; (void)v; (void)hv; (void)dv; (void)e; (void)s; (void)c; (void)g;
}
void __hipRegisterFunction(void **h, const void *host, char *f, const char *name, unsigned t, void *a, void *b, void *c,
                           void *d, int *w)
{
    (void)h; (void)f; (void)t; (void)a; (void)b; (void)c; (void)d; (void)w;
    if (n_funcs < MAX_FUNCS) { funcs[n_funcs].host = host; funcs[n_funcs++].name = name; }
}

static __thread struct { dim3_t g, b; size_t lds; void *s; } config;
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t lds, void *s)
{
    config.g = g; config.b = b; config.lds = lds; config.s = s;
    return 0;
}
int __hipPopCallConfiguration(dim3_t *g, dim3_t *b, size_t *lds, void **s)
{
    *g = config.g; *b = config.b; *lds = config.lds; *s = config.s;
    return 0;
}
int hipLaunchKernel(const void *f, dim3_t g, dim3_t b, void **args, size_t lds, void *s)
{
    (void)args; (void)lds; (void)s;
    const char *name = "?";
    for (int i = 0; i < n_funcs; ++i)
        if (funcs[i].host == f) name = funcs[i].name;
    if (fail_times > 0 && strstr(name, fail_name)) {
        --fail_times;
        return last_error = 719;
    }
    if (n_log < MAX_LOG) { log_[n_log].name = name; log_[n_log].grid = g.x; log_[n_log++].threads = b.x; }
    return 0;
}
int hipGetLastError(void) { const int e = last_error; last_error = 0; return e; }
const char *hipGetErrorString(int e) { return e ? "recorded failure" : "no error"; }

int hipMalloc(void **p, size_t n) { *p = calloc(1, n ? n : 1); return *p ? 0 : 2; }
int hipFree(void *p) { free(p); return 0; }
int hipMemcpy(void *d, const void *s, size_t n, int k) { (void)k; memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *st) { (void)k; (void)st; memcpy(d, s, n); return 0; }
int hipMemset(void *d, int v, size_t n) { memset(d, v, n); return 0; }
int hipGetSymbolAddress(void **p, const void *sym) { (void)sym; *p = calloc(1, 65 << 20); return *p ? 0 : 2; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipSetDevice(int d) { (void)d; return 0; }
int hipDeviceGetAttribute(int *v, int a, int d) { (void)a; (void)d; *v = 256; return 0; }
int hipGetDevicePropertiesR0600(void *p, int d) { (void)p; (void)d; return 1; }
int hipDeviceSynchronize(void) { return 0; }
int hipStreamSynchronize(void *s) { (void)s; return 0; }
int hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; *s = NULL; return 0; }
int hipStreamDestroy(void *s) { (void)s; return 0; }
int hipStreamBeginCapture(void *s, int m) { (void)s; (void)m; return 0; }
int hipStreamEndCapture(void *s, void **g) { (void)s; *g = NULL; return 0; }
int hipGraphInstantiate(void **e, void *g, void *n, char *b, size_t z) { (void)g; (void)n; (void)b; (void)z; *e = NULL; return 0; }
int hipGraphLaunch(void *e, void *s) { (void)e; (void)s; return 0; }
int hipGraphExecDestroy(void *e) { (void)e; return 0; }
int hipGraphDestroy(void *g) { (void)g; return 0; }
int hipFuncSetAttribute(const void *f, int a, int v) { (void)f; (void)a; (void)v; return 0; }
int hipEventCreate(void **e) { *e = malloc(1); return 0; }
int hipEventDestroy(void *e) { free(e); return 0; }
int hipEventRecord(void *e, void *s) { (void)e; (void)s; return 0; }
int hipEventSynchronize(void *e) { (void)e; return 0; }
int hipEventElapsedTime(float *ms, void *a, void *b)
{
    (void)a; (void)b;
    noise = noise * 1664525u + 1013904223u;
    *ms = 1.0f + 0.01f * (float)(noise >> 8) / 16777216.0f;
    return 0;
}
