/* The HIP runtime calls of the library, on host memory: allocations are
 * malloc's (up to a limit the test sets), copies memcpy's, a kernel launch
 * only records the kernel's name, grid, block and LDS bytes.  Loaded with
 * RTLD_GLOBAL before the library, it takes the runtime's place in a process
 * without a GPU, so that mesh setup, launch plans and failed allocations can
 * be tested there.  Streams and events are dummies. */
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;
#define OK 0
#define OUT_OF_MEMORY 2

static long long g_used, g_limit = -1; /* bytes; -1: no limit */
static int g_allocs, g_error; /* the error the next hipGetLastError returns */
void host_hip_limit(long long bytes) { g_limit = bytes; }
long long host_hip_used(void) { return g_used; }
int host_hip_allocs(void) { return g_allocs; }

int hipMalloc(void **p, size_t n) {
  *p = NULL;
  if (g_limit >= 0 && g_used + (long long)n > g_limit) return g_error = OUT_OF_MEMORY;
  size_t *b = aligned_alloc(256, (n + 256 + 255) / 256 * 256);
  if (!b) return g_error = OUT_OF_MEMORY;
  b[0] = n;
  g_used += (long long)n;
  ++g_allocs;
  *p = (char *)b + 256;
  return OK;
}
int hipFree(void *p) {
  if (!p) return OK;
  size_t *b = (size_t *)((char *)p - 256);
  g_used -= (long long)b[0];
  free(b);
  return OK;
}
int hipMallocAsync(void **p, size_t n, void *s) { (void)s; return hipMalloc(p, n); }
int hipFreeAsync(void *p, void *s) { (void)s; return hipFree(p); }
int hipHostMalloc(void **p, size_t n, unsigned f) { (void)f; *p = malloc(n); return *p ? OK : OUT_OF_MEMORY; }
int hipHostFree(void *p) { free(p); return OK; }
int hipMemcpy(void *d, const void *s, size_t n, int k) { (void)k; memcpy(d, s, n); return OK; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *st) { (void)k; (void)st; memcpy(d, s, n); return OK; }
int hipGetDevice(int *d) { *d = 0; return OK; }
int hipSetDevice(int d) { (void)d; return OK; }
int hipDeviceSynchronize(void) { return OK; }
int hipGetLastError(void) { const int e = g_error; g_error = OK; return e; }
const char *hipGetErrorString(int e) { return e == OUT_OF_MEMORY ? "out of memory" : "error"; }
int hipDeviceGetAttribute(int *v, int a, int d) { (void)a; (void)d; *v = 256; return OK; } /* compute units */
int hipFuncSetAttribute(const void *f, int a, int v) { (void)f; (void)a; (void)v; return OK; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int b, size_t s) {
  (void)f; (void)b; (void)s; *n = 1; return OK;
}
int hipGetSymbolAddress(void **p, const void *s) { (void)s; static char buf[1 << 20]; *p = buf; return OK; }

/* events: a clock that every launch moves on by one millisecond, or by a
 * hundred for a kernel whose name holds `name` (host_hip_slow) */
static double g_clock;
static char g_slow[128];
void host_hip_slow(const char *name) { snprintf(g_slow, sizeof g_slow, "%s", name); }
int hipEventCreate(void **e) { *e = calloc(1, sizeof(double)); return OK; }
int hipEventCreateWithFlags(void **e, unsigned f) { (void)f; return hipEventCreate(e); }
int hipEventDestroy(void *e) { free(e); return OK; }
int hipEventRecord(void *e, void *s) { (void)s; *(double *)e = g_clock; return OK; }
int hipEventSynchronize(void *e) { (void)e; return OK; }
int hipEventQuery(void *e) { (void)e; return OK; }
int hipEventElapsedTime(float *ms, void *a, void *b) { *ms = (float)(*(double *)b - *(double *)a); return OK; }
int hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; *s = calloc(1, 1); return OK; }
int hipStreamDestroy(void *s) { free(s); return OK; }
int hipStreamSynchronize(void *s) { (void)s; return OK; }
int hipStreamWaitEvent(void *s, void *e, unsigned f) { (void)s; (void)e; (void)f; return OK; }

/* kernels: names by host function, and the list of launches */
static struct { const void *fn; char name[160]; } g_kern[4096];
static int g_nkern;
void **__hipRegisterFatBinary(const void *d) { (void)d; static void *h; return &h; }
void __hipUnregisterFatBinary(void **h) { (void)h; }
void __hipRegisterVar(void **h, void *v, char *a, char *b, int e, size_t n, int c, int g) {
  (void)h; (void)v; (void)a; (void)b; (void)e; (void)n; (void)c; (void)g;
}
void __hipRegisterFunction(void **h, const void *fn, char *dev, const char *name, unsigned t, void *a,
                           void *b, void *c, void *d, int *w) {
  (void)h; (void)dev; (void)t; (void)a; (void)b; (void)c; (void)d; (void)w;
  if (g_nkern < 4096) {
    g_kern[g_nkern].fn = fn;
    snprintf(g_kern[g_nkern++].name, sizeof g_kern[0].name, "%s", name);
  }
}
static struct { dim3_t g, b; size_t l; void *s; } g_cfg;
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t l, void *s) {
  g_cfg.g = g; g_cfg.b = b; g_cfg.l = l; g_cfg.s = s;
  return OK;
}
int __hipPopCallConfiguration(dim3_t *g, dim3_t *b, size_t *l, void **s) {
  *g = g_cfg.g; *b = g_cfg.b; *l = g_cfg.l; *s = g_cfg.s;
  return OK;
}
static char g_log[1 << 20];
static size_t g_len;
void host_hip_clear(void) { g_len = 0; g_log[0] = 0; }
const char *host_hip_log(void) { return g_log; }
int hipLaunchKernel(const void *fn, dim3_t g, dim3_t b, void **args, size_t lds, void *s) {
  (void)args; (void)s;
  const char *name = "?";
  for (int i = 0; i < g_nkern; ++i)
    if (g_kern[i].fn == fn) name = g_kern[i].name;
  g_clock += g_slow[0] && strstr(name, g_slow) ? 100.0 : 1.0;
  if (g_len + 512 < sizeof g_log)
    g_len += (size_t)snprintf(g_log + g_len, 512, "%s %u %u %zu\n", name, g.x, b.x, lds);
  return OK;
}
