// A HIP runtime that runs nothing, for tests of the library's host side where
// there is no GPU: device memory is addresses that nothing reads, copies to the
// host give zeros, and every launch, asynchronous copy and synchronisation is
// shown to the test.  Loaded before the library, with its symbols global, it
// takes the place of the runtime the library was linked against.
#include <hip/hip_runtime_api.h>
#include <stdlib.h>
#include <string.h>

typedef int (*launch_fn)(const char *kernel, const uint32_t *grid, uint32_t threads, size_t lds, void **args);
typedef void (*event_fn)(const char *what, const void *src, size_t bytes);
static launch_fn on_launch;
static event_fn on_event;
void stand_in_watch(launch_fn l, event_fn e) {
  on_launch = l;
  on_event = e;
}

static struct {
  const void *host;
  const char *name;
} kernels[256];
static int n_kernels;
static hipError_t last;
static uintptr_t next = (uintptr_t)1 << 44;

void **__hipRegisterFatBinary(const void *data) {
  static void *module;
  (void)data;
  return &module;
}
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterVar(void) {}
void __hipRegisterFunction(void **m, const void *host, char *device, const char *name, unsigned limit, void *t, void *b,
                           void *bd, void *gd, int *w) {
  (void)m, (void)device, (void)limit, (void)t, (void)b, (void)bd, (void)gd, (void)w;
  if (n_kernels < 256) kernels[n_kernels].host = host, kernels[n_kernels++].name = name;
}
static struct {
  dim3 g, b;
  size_t lds;
  hipStream_t s;
} call;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s) {
  call.g = g, call.b = b, call.lds = lds, call.s = s;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, hipStream_t *s) {
  *g = call.g, *b = call.b, *lds = call.lds, *s = call.s;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t lds, hipStream_t s) {
  const uint32_t grid[3] = {g.x, g.y, g.z};
  (void)s;
  for (int i = 0; i < n_kernels; i++)
    if (kernels[i].host == f && on_launch) last = (hipError_t)on_launch(kernels[i].name, grid, b.x * b.y * b.z, lds, args);
  return last;
}
hipError_t hipGetLastError(void) {
  const hipError_t e = last;
  last = hipSuccess;
  return e;
}
const char *hipGetErrorString(hipError_t e) { return e == hipSuccess ? "no error" : "an error of the stand-in"; }

static hipError_t take(void **p, size_t n) {
  *p = (void *)next;
  next += (n + 511) & ~(size_t)255;
  return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n) { return take(p, n); }
hipError_t hipMallocAsync(void **p, size_t n, hipStream_t s) { return (void)s, take(p, n); }
hipError_t hipMallocFromPoolAsync(void **p, size_t n, hipMemPool_t m, hipStream_t s) { return (void)m, (void)s, take(p, n); }
hipError_t hipFree(void *p) { return (void)p, hipSuccess; }
hipError_t hipFreeAsync(void *p, hipStream_t s) { return (void)p, (void)s, hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned f) { return (void)f, (*p = malloc(n)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipHostFree(void *p) { return free(p), hipSuccess; }
hipError_t hipMemPoolCreate(hipMemPool_t *m, const hipMemPoolProps *p) { return (void)p, *m = (hipMemPool_t)next, hipSuccess; }
hipError_t hipMemPoolSetAttribute(hipMemPool_t m, hipMemPoolAttr a, void *v) { return (void)m, (void)a, (void)v, hipSuccess; }
hipError_t hipMemGetAddressRange(hipDeviceptr_t *base, size_t *n, hipDeviceptr_t p) {
  if ((uintptr_t)p < (uintptr_t)1 << 44) return hipErrorInvalidValue;
  *base = (hipDeviceptr_t)((uintptr_t)1 << 44);
  *n = (size_t)1 << 45;
  return hipSuccess;
}
static hipError_t copy(void *dst, size_t n, hipMemcpyKind k) {
  if (k == hipMemcpyDeviceToHost && n <= (size_t)1 << 20) memset(dst, 0, n);
  return hipSuccess;
}
hipError_t hipMemcpy(void *dst, const void *src, size_t n, hipMemcpyKind k) { return (void)src, copy(dst, n, k); }
hipError_t hipMemcpyAsync(void *dst, const void *src, size_t n, hipMemcpyKind k, hipStream_t s) {
  (void)s;
  if (on_event) on_event(k == hipMemcpyHostToDevice ? "copy in" : "copy out", src, n);
  return copy(dst, n, k);
}
hipError_t hipMemset(void *p, int v, size_t n) { return (void)p, (void)v, (void)n, hipSuccess; }
hipError_t hipMemsetAsync(void *p, int v, size_t n, hipStream_t s) { return (void)s, hipMemset(p, v, n); }
hipError_t hipStreamSynchronize(hipStream_t s) {
  if (on_event) on_event("wait", s, 0);
  return hipSuccess;
}
hipError_t hipDeviceSynchronize(void) { return hipStreamSynchronize(0); }
hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipSetDevice(int d) { return d ? hipErrorInvalidDevice : hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int d) {
  (void)d;
  *v = a == hipDeviceAttributeMaxSharedMemoryPerBlock ? 160 * 1024 : (a == hipDeviceAttributeMultiprocessorCount ? 256 : 0);
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *symbol) { return (void)symbol, take(p, 256); }
hipError_t hipEventCreate(hipEvent_t *e) { return take((void **)e, 1); }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned f) { return (void)f, take((void **)e, 1); }
hipError_t hipEventDestroy(hipEvent_t e) { return (void)e, hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { return (void)e, (void)s, hipSuccess; }
hipError_t hipEventQuery(hipEvent_t e) { return (void)e, hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t e) { return (void)e, hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t a, hipEvent_t b) { return (void)a, (void)b, *ms = 1.0f, hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned f) { return (void)f, take((void **)s, 1); }
hipError_t hipStreamDestroy(hipStream_t s) { return (void)s, hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned f) { return (void)s, (void)e, (void)f, hipSuccess; }
