/* A HIP runtime without a device, loaded in front of the real one: device
 * memory is host memory nobody reads, kernel launches do nothing.  hipMalloc
 * refuses more than FAKE_HIP_LARGEST bytes at once; every allocation is
 * reported on standard output. */
#include <stdio.h>
#include <stdlib.h>

typedef struct {
  unsigned x, y, z;
} dim3;

enum { kOk = 0, kOutOfMemory = 2 };

static int take(const char *call, void **p, size_t n) {
  const char *s = getenv("FAKE_HIP_LARGEST");
  const int ok = !s || n <= strtoull(s, 0, 10);
  *p = ok ? aligned_alloc(256, (n + 255) / 256 * 256) : 0;
  printf("%s %zu %s\n", call, n, ok ? "ok" : "refused");
  fflush(stdout);
  return ok ? kOk : kOutOfMemory;
}

int hipGetDeviceCount(int *n) { return *n = 1, kOk; }
int hipGetDevice(int *d) { return *d = 0, kOk; }
int hipSetDevice(int d) { return d ? 101 : kOk; }
int hipDeviceSynchronize(void) { return kOk; }
int hipGetLastError(void) { return kOk; }
int hipMalloc(void **p, size_t n) { return take("malloc", p, n); }
int hipMallocAsync(void **p, size_t n, void *s) { return (void)s, take("pool", p, n); }
int hipFree(void *p) { return free(p), kOk; }
int hipFreeAsync(void *p, void *s) { return (void)s, free(p), kOk; }
int hipMemset(void *p, int v, size_t n) { return (void)p, (void)v, (void)n, kOk; }
int hipThreadExchangeStreamCaptureMode(int *mode) { return (void)mode, kOk; }
int hipStreamIsCapturing(void *s, int *status) { return (void)s, *status = 0, kOk; }
int hipGetDevicePropertiesR0600(void *prop, int d) {
  /* name, uuid, luid, luidDeviceNodeMask, totalGlobalMem: 288 GiB at byte 288 */
  (void)d;
  for (int i = 0; i < 1472; ++i) ((char *)prop)[i] = 0;
  *(size_t *)((char *)prop + 288) = (size_t)288 << 30;
  return kOk;
}
int hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t lds, void *s) {
  return (void)f, (void)grid, (void)block, (void)args, (void)lds, (void)s, kOk;
}
