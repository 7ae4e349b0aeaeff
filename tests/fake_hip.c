/* A stand-in for the HIP runtime that records what the library's host code asks of it: device memory is host memory,
 * kernels do not run.  Built as libamdhip64.so.7 and loaded before the library, which then takes its calls here. */
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3;
typedef struct { const void *host; char name[512]; } kernel_t;

static kernel_t kernels[4096];
static int nkernels;
static char *text;
static size_t used, room;
static size_t fail_above = (size_t)-1;
static uint64_t prepass[64];          /* what k_prepass leaves in its counters */

static void note(const char *what, const char *arg, long long value) {
    if (room - used < 1024) { room = 2 * room + 65536; text = realloc(text, room); }
    used += (size_t)snprintf(text + used, 1024, "%s %s %lld\n", what, arg, value);
}
static const char *name_of(const void *f) {
    for (int i = 0; i < nkernels; ++i) if (kernels[i].host == f) return kernels[i].name;
    return "?";
}

const char *fake_text(void) { note("end", "-", 0); return text; }
void fake_reset(size_t limit) { used = 0; fail_above = limit; memset(prepass, 0, sizeof prepass); }
void fake_prepass(int word, uint64_t value) { prepass[word] = value; }

void **__hipRegisterFatBinary(const void *data) { static void *h; (void)data; return &h; }
void __hipUnregisterFatBinary(void **h) { (void)h; }
void __hipRegisterVar(void **h, void *v, char *hn, char *dn, int e, size_t s, int c, int g) { (void)h; (void)v; (void)hn; (void)dn; (void)e; (void)s; (void)c; (void)g; }
void __hipRegisterFunction(void **h, const void *host, char *dev, const char *name, unsigned n, void *a, void *b, void *c, void *d, int *e) {
    (void)h; (void)dev; (void)n; (void)a; (void)b; (void)c; (void)d; (void)e;
    if (nkernels < 4096) { kernels[nkernels].host = host; snprintf(kernels[nkernels++].name, 512, "%s", name); }
}
static dim3 cfg_grid, cfg_block; static size_t cfg_lds; static void *cfg_stream;
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t l, void *s) { cfg_grid = g; cfg_block = b; cfg_lds = l; cfg_stream = s; return 0; }
int __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *l, void **s) { *g = cfg_grid; *b = cfg_block; *l = cfg_lds; *s = cfg_stream; return 0; }
int hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t lds, void *s) {
    const char *name = name_of(f);
    (void)b; (void)s; (void)g;
    note("launch", name, (long long)lds);
    if (strstr(name, "k_prepass")) memcpy(*(void **)args[6], prepass, 32 * 8);
    return 0;
}
int hipFuncSetAttribute(const void *f, int attr, int value) { (void)attr; note("attribute", name_of(f), value); return 0; }
int hipMalloc(void **p, size_t n) { return hipMallocAsync(p, n, 0); }
int hipMallocAsync(void **p, size_t n, void *s) {
    (void)s;
    note(n > fail_above ? "refused" : "malloc", "-", (long long)n);
    if (n > fail_above) return 2;
    return (*p = calloc(1, n)) ? 0 : 2;
}
int hipFree(void *p) { free(p); return 0; }
int hipFreeAsync(void *p, void *s) { (void)s; free(p); note("free", "-", 0); return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *st) { (void)st; memcpy(d, s, n); note("copy", "-", kind); return 0; }
int hipMemsetAsync(void *d, int v, size_t n, void *s) { (void)s; memset(d, v, n); return 0; }
int hipStreamSynchronize(void *s) { (void)s; note("wait", "-", 0); return 0; }
int hipDeviceSynchronize(void) { return 0; }
int hipStreamIsCapturing(void *s, int *c) { (void)s; *c = 0; return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipGetLastError(void) { return 0; }
int hipGetSymbolAddress(void **p, const void *s) { static double buf[1 << 19]; (void)s; *p = buf; return 0; }
int hipEventCreateWithFlags(void **e, unsigned f) { (void)f; *e = malloc(1); return 0; }
int hipEventDestroy(void *e) { free(e); return 0; }
int hipEventRecord(void *e, void *s) { (void)e; (void)s; note("record", "-", 0); return 0; }
int hipEventSynchronize(void *e) { (void)e; return 0; }
int hipEventElapsedTime(float *ms, void *a, void *b) { (void)a; (void)b; *ms = 1.0f; return 0; }
