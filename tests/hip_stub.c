/* The HIP runtime calls of the library on host memory, for CPU tests of its host drivers: allocations can be
 * made to fail, kernel launches do nothing, and a copy of the CG scalars to the host reads as converged. */
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

enum { OK = 0, OUT_OF_MEMORY = 2, D2H = 2, MAX = 1 << 16 };

static void *g_ptr[MAX];
static size_t g_size[MAX];
static int g_n = 0;
static long g_fail_at = 0, g_failed = 0;   /* fail the g_fail_at-th allocation from now (0: none) */

void stub_fail_at(long k) { g_fail_at = k, g_failed = 0; }
long stub_failed(void) { return g_failed; }
long stub_live(void) { return g_n; }
size_t stub_live_bytes(void) {
  size_t s = 0;
  for (int k = 0; k < g_n; ++k) s += g_size[k];
  return s;
}

static int give(void **p, size_t n) {
  if (g_fail_at > 0 && --g_fail_at == 0) {
    g_failed = 1;
    return OUT_OF_MEMORY;
  }
  *p = calloc(1, n);
  g_ptr[g_n] = *p;
  g_size[g_n++] = n;
  return OK;
}
static int take(void *p) {
  for (int k = 0; k < g_n; ++k)
    if (g_ptr[k] == p) {
      free(p);
      --g_n;
      g_ptr[k] = g_ptr[g_n];
      g_size[k] = g_size[g_n];
      return OK;
    }
  return 1;
}
int hipMalloc(void **p, size_t n) { return give(p, n); }
int hipHostMalloc(void **p, size_t n, unsigned f) { return give(p, n); }
int hipFree(void *p) { return take(p); }
int hipHostFree(void *p) { return take(p); }
int hipMemset(void *p, int v, size_t n) { return memset(p, v, n), OK; }
int hipMemcpy(void *d, const void *s, size_t n, int kind) { return memcpy(d, s, n), OK; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *stream) {
  memcpy(d, s, n);
  /* eight doubles, then done, iters, breakdown and padding */
  if (kind == D2H && (n == 80 || n == 160))
    for (size_t k = 0; k < n; k += 80) ((int32_t *)((char *)d + k))[16] = 1;
  return OK;
}
int hipMemcpyToSymbol(const void *sym, const void *s, size_t n, size_t o, int kind) { return OK; }
int hipGetSymbolAddress(void **p, const void *sym) {
  static char somewhere[1 << 20];
  *p = somewhere;
  return OK;
}
int hipGetDevice(int *d) { return *d = 0, OK; }
int hipDeviceSynchronize(void) { return OK; }
int hipGetLastError(void) { return OK; }
const char *hipGetErrorString(int e) { return e == OUT_OF_MEMORY ? "out of memory" : "error"; }
int hipLaunchKernel(const void *f, ...) { return OK; }
int hipStreamCreateWithFlags(void **s, unsigned f) { return *s = (void *)g_ptr, OK; }
int hipStreamDestroy(void *s) { return OK; }
int hipStreamSynchronize(void *s) { return OK; }
int hipStreamIsCapturing(void *s, int *c) { return *c = 0, OK; }
int hipStreamBeginCapture(void *s, int mode) { return OK; }
int hipStreamEndCapture(void *s, void **g) { return *g = (void *)g_ptr, OK; }
int hipGraphInstantiate(void **x, void *g, void *n, char *b, size_t z) { return *x = (void *)g_ptr, OK; }
int hipGraphLaunch(void *x, void *s) { return OK; }
int hipGraphDestroy(void *g) { return OK; }
int hipGraphExecDestroy(void *x) { return OK; }
void **__hipRegisterFatBinary(const void *d) {
  static void *h;
  return &h;
}
void __hipUnregisterFatBinary(void **h) {}
void __hipRegisterFunction(void) {}
void __hipRegisterVar(void) {}
int __hipPushCallConfiguration(void) { return OK; }
int __hipPopCallConfiguration(void) { return OK; }
