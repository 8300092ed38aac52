/* A stand-in for the HIP runtime calls of libexageo.so on a machine without a
 * GPU: device memory is zeroed host memory, kernels are not run, and every
 * runtime call is written to the file named by FAKEHIP_LOG.  Loaded with
 * RTLD_GLOBAL before the library, so that its undefined hip* symbols bind
 * here. */
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3;

static FILE *out;
static struct { const void *host; const char *name; } kern[4096];
static int nkern;
static uintptr_t handles = 1;

void fakehip_mark(const char *what) {
  if (!out) out = fopen(getenv("FAKEHIP_LOG"), "w");
  fprintf(out, "%s\n", what);
  fflush(out);
}

static int handle(void **p, const char *what) {
  char line[64];
  *p = (void *)(handles++);
  snprintf(line, sizeof line, "%s %p", what, *p);
  fakehip_mark(line);
  return 0;
}
static int memory(void **p, size_t n, const char *what) {
  *p = calloc(n, 1);
  fakehip_mark(what);
  return *p ? 0 : 2;
}

int hipGetDeviceCount(int *n) { *n = 1; return 0; }
int hipSetDevice(int d) { (void)d; return 0; }
int hipDeviceSynchronize(void) { return 0; }
int hipGetLastError(void) { return 0; }
const char *hipGetErrorString(int e) { (void)e; return "fake"; }
int hipMalloc(void **p, size_t n) { return memory(p, n, "hipMalloc"); }
int hipHostMalloc(void **p, size_t n, unsigned f) { (void)f; return memory(p, n, "hipHostMalloc"); }
int hipGetSymbolAddress(void **p, const void *s) { (void)s; return memory(p, (size_t)128 << 20, "hipGetSymbolAddress"); }
int hipFree(void *p) { free(p); fakehip_mark("hipFree"); return 0; }
int hipHostFree(void *p) { free(p); fakehip_mark("hipHostFree"); return 0; }
int hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; return handle(s, "hipStreamCreateWithFlags"); }
int hipStreamDestroy(void *s) { (void)s; fakehip_mark("hipStreamDestroy"); return 0; }
int hipStreamSynchronize(void *s) { (void)s; fakehip_mark("hipStreamSynchronize"); return 0; }
int hipStreamWaitEvent(void *s, void *e, unsigned f) { (void)s; (void)e; (void)f; fakehip_mark("hipStreamWaitEvent"); return 0; }
int hipEventCreate(void **e) { return handle(e, "hipEventCreate"); }
int hipEventCreateWithFlags(void **e, unsigned f) { (void)f; return handle(e, "hipEventCreateWithFlags"); }
int hipEventDestroy(void *e) { (void)e; fakehip_mark("hipEventDestroy"); return 0; }
int hipEventRecord(void *e, void *s) {
  char line[64];
  snprintf(line, sizeof line, "hipEventRecord %p %p", e, s);
  fakehip_mark(line);
  return 0;
}
int hipEventSynchronize(void *e) { (void)e; return 0; }
int hipEventElapsedTime(float *ms, void *a, void *b) { (void)a; (void)b; *ms = 0; return 0; }
int hipMemcpy(void *d, const void *s, size_t n, int k) { (void)k; memcpy(d, s, n); fakehip_mark("hipMemcpy"); return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *st) {
  (void)k; (void)st;
  memcpy(d, s, n);
  fakehip_mark("hipMemcpyAsync");
  return 0;
}

/* kernel registration and launches */
void **__hipRegisterFatBinary(const void *data) { (void)data; return (void **)&kern; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterFunction(void **m, const void *host, char *dev, const char *name, unsigned lim, void *t, void *b,
                           void *bd, void *gd, int *w) {
  (void)m; (void)dev; (void)lim; (void)t; (void)b; (void)bd; (void)gd; (void)w;
  kern[nkern].host = host;
  kern[nkern++].name = name;
}
void __hipRegisterVar(void **m, void *v, char *hv, char *dv, int ext, size_t n, int c, int g) {
  (void)m; (void)v; (void)hv; (void)dv; (void)ext; (void)n; (void)c; (void)g;
}
static struct { dim3 grid, block; size_t shm; void *stream; } cfg;
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shm, void *stream) {
  cfg.grid = grid, cfg.block = block, cfg.shm = shm, cfg.stream = stream;
  return 0;
}
int __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shm, void **stream) {
  *grid = cfg.grid, *block = cfg.block, *shm = cfg.shm, *stream = cfg.stream;
  return 0;
}
int hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t shm, void *stream) {
  char line[512];
  (void)args;
  for (int i = 0; i < nkern; ++i)
    if (kern[i].host == f) {
      snprintf(line, sizeof line, "launch %s %u %u %zu %p", kern[i].name, grid.x, block.x, shm, stream);
      fakehip_mark(line);
      return 0;
    }
  return 98;
}
