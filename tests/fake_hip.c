/* A stand-in for the HIP runtime with two devices, preloaded by
   tests/test_current_device_cpu.py: device memory is host memory that
   remembers its device, kernels do nothing, and a launch, copy or allocation
   that mixes devices is reported.  Only what the library's table and batch
   calls use is here. */
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#define MAX_ALLOCS 4096
static __thread int cur = 0;
static struct { char* p; size_t n; int dev; } allocs[MAX_ALLOCS];
static int n_allocs = 0;
int fake_wrong = 0;    /* launches on a device that does not own their memory */
int fake_launches = 0;
int fake_mallocs[2] = {0, 0};

static int owner(const void* q) {
  for (int i = 0; i < n_allocs; ++i)
    if ((const char*)q >= allocs[i].p && (const char*)q < allocs[i].p + allocs[i].n) return allocs[i].dev;
  return -1;
}
int hipGetDevice(int* d) { *d = cur; return 0; }
int hipSetDevice(int d) { if (d < 0 || d > 1) return 101; cur = d; return 0; }
int hipGetLastError(void) { return 0; }
int hipMalloc(void** p, size_t n) {
  if (n_allocs == MAX_ALLOCS) return 2;
  *p = calloc(1, n ? n : 1);
  if (!*p) return 2;
  allocs[n_allocs].p = *p; allocs[n_allocs].n = n; allocs[n_allocs++].dev = cur;
  ++fake_mallocs[cur];
  return 0;
}
int hipFree(void* p) {
  for (int i = 0; i < n_allocs; ++i)
    if (allocs[i].p == p) { allocs[i].p = 0; allocs[i].n = 0; free(p); }
  return 0;
}
int hipHostMalloc(void** p, size_t n, unsigned f) { (void)f; *p = calloc(1, n); return *p ? 0 : 2; }
int hipHostFree(void* p) { free(p); return 0; }
int hipMemcpy(void* d, const void* s, size_t n, int k) { (void)k; memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int k, void* st) { (void)st; return hipMemcpy(d, s, n, k); }
int hipDeviceSynchronize(void) { return 0; }
int hipStreamSynchronize(void* s) { (void)s; return 0; }
int hipDeviceGetAttribute(int* v, int a, int d) { (void)a; (void)d; *v = 256; return 0; }

typedef struct { uint32_t x, y, z; } dim3_;
static dim3_ pg, pb;
static size_t psh;
static void* pst;
int __hipPushCallConfiguration(dim3_ g, dim3_ b, size_t sh, void* st) { pg = g; pb = b; psh = sh; pst = st; return 0; }
int __hipPopCallConfiguration(dim3_* g, dim3_* b, size_t* sh, void** st) { *g = pg; *b = pb; *sh = psh; *st = pst; return 0; }
/* the kernels under test take a device pointer first */
int hipLaunchKernel(const void* f, dim3_ g, dim3_ b, void** args, size_t sh, void* st) {
  (void)f; (void)g; (void)b; (void)sh; (void)st;
  ++fake_launches;
  const int dev = owner(*(void**)args[0]);
  if (dev >= 0 && dev != cur) { ++fake_wrong; }
  return 0;
}
