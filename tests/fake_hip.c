/* The part of the HIP runtime that libadmm.so calls, on host memory and without
 * a device: allocations against a budget, copies done at once, kernels not run
 * but their launches recorded. For the tests of what the host code allocates
 * and launches; loaded with RTLD_GLOBAL before libadmm.so. */
#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_;
enum { OUT_OF_MEMORY = 2, MAX_BLOCKS = 4096 };

static size_t budget = (size_t)-1, used = 0, largest = 0, lds_most = 0;
static struct { void *p; size_t n; } blocks[MAX_BLOCKS];
static int last_error = 0, launches = 0;
static uint64_t shape_hash = 0;
static double event_ms = 1.0, event_factor = 1.0;

void fake_reset(size_t b) {
  budget = b;
  largest = lds_most = 0;
  launches = 0;
  shape_hash = 0;
}
/* the next timing, and by what factor each one after it is longer */
void fake_event_ms(double ms, double factor) {
  event_ms = ms;
  event_factor = factor;
}
/* of the launches' grids, blocks and LDS sizes, in order */
uint64_t fake_shape_hash(void) { return shape_hash; }
size_t fake_used(void) { return used; }
size_t fake_largest(void) { return largest; }
size_t fake_lds_most(void) { return lds_most; }
int fake_launches(void) { return launches; }

int hipMalloc(void **p, size_t n) {
  if (n > budget || used > budget - n) return last_error = OUT_OF_MEMORY;
  for (int k = 0; k < MAX_BLOCKS; ++k)
    if (!blocks[k].p) {
      if (posix_memalign(p, 256, n ? n : 1)) return last_error = OUT_OF_MEMORY;
      memset(*p, 0, n);
      blocks[k].p = *p;
      blocks[k].n = n;
      used += n;
      if (n > largest) largest = n;
      return 0;
    }
  return last_error = OUT_OF_MEMORY;
}
int hipFree(void *p) {
  for (int k = 0; p && k < MAX_BLOCKS; ++k)
    if (blocks[k].p == p) {
      used -= blocks[k].n;
      blocks[k].p = NULL;
      free(p);
      return 0;
    }
  return p ? 1 : 0;
}
int hipGetLastError(void) {
  int e = last_error;
  last_error = 0;
  return e;
}
int hipMemcpy(void *d, const void *s, size_t n, int kind) { return memcpy(d, s, n), (void)kind, 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *st) {
  return memcpy(d, s, n), (void)kind, (void)st, 0;
}
int hipMemset(void *d, int v, size_t n) { return memset(d, v, n), 0; }
int hipGetDevice(int *d) { return *d = 0, 0; }
int hipGetDeviceCount(int *n) { return *n = 1, 0; }
int hipGetSymbolAddress(void **p, const void *s) { return *p = NULL, (void)s, 1; }
int hipStreamSynchronize(void *s) { return (void)s, 0; }
int hipStreamCreateWithFlags(void **s, unsigned f) { return *s = NULL, (void)f, 0; }
int hipStreamDestroy(void *s) { return (void)s, 0; }
int hipStreamBeginCapture(void *s, int m) { return (void)s, (void)m, 0; }
int hipStreamEndCapture(void *s, void **g) { return (void)s, *g = NULL, 0; }
int hipGraphInstantiate(void **e, void *g, void **n, char *b, size_t z) {
  return *e = (void *)1, (void)g, (void)n, (void)b, (void)z, 0;
}
int hipGraphLaunch(void *e, void *s) { return (void)e, (void)s, 0; }
int hipGraphDestroy(void *g) { return (void)g, 0; }
int hipGraphExecDestroy(void *e) { return (void)e, 0; }
int hipEventCreate(void **e) { return *e = (void *)1, 0; }
int hipEventDestroy(void *e) { return (void)e, 0; }
int hipEventRecord(void *e, void *s) { return (void)e, (void)s, 0; }
int hipEventSynchronize(void *e) { return (void)e, 0; }
int hipEventElapsedTime(float *ms, void *a, void *b) {
  *ms = (float)event_ms;
  event_ms *= event_factor;
  return (void)a, (void)b, 0;
}

void **__hipRegisterFatBinary(const void *data) { return (void)data, (void **)1; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterFunction(void **m, const void *host, char *dev, const char *name, unsigned lim,
                           void *tid, void *bid, void *bd, void *gd, int *ws) {
  (void)m, (void)host, (void)dev, (void)name, (void)lim, (void)tid, (void)bid, (void)bd, (void)gd, (void)ws;
}
void __hipRegisterVar(void **m, void *v, char *h, char *d, int e, size_t n, int c, int g) {
  (void)m, (void)v, (void)h, (void)d, (void)e, (void)n, (void)c, (void)g;
}
static struct { dim3_ g, b; size_t lds; void *st; } call;
int __hipPushCallConfiguration(dim3_ g, dim3_ b, size_t lds, void *st) {
  call.g = g, call.b = b, call.lds = lds, call.st = st;
  return 0;
}
int __hipPopCallConfiguration(dim3_ *g, dim3_ *b, size_t *lds, void **st) {
  *g = call.g, *b = call.b, *lds = call.lds, *st = call.st;
  return 0;
}
int hipLaunchKernel(const void *f, dim3_ g, dim3_ b, void **args, size_t lds, void *st) {
  const uint64_t w[7] = {g.x, g.y, g.z, b.x, b.y, b.z, lds};
  (void)f, (void)args, (void)st;
  ++launches;
  for (int k = 0; k < 7; ++k) shape_hash = (shape_hash ^ w[k]) * 0x100000001b3ull;
  if (lds > lds_most) lds_most = lds;
  return 0;
}
