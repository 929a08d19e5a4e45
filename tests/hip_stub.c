/* A stand-in for the HIP runtime, preloaded by test_launches_host.py: the
 * library's host code runs on a machine without a GPU, every kernel launch is
 * written to the log (HIP_STUB_LOG: kernel, grid, block, current device) and
 * none is executed.  Device pointers are made up, so copies do nothing.
 * A launch of 2^32 threads or more in a dimension is refused, as HIP documents.
 * The lineage walk leaves its summary in host memory: HIP_STUB_LINEAGE
 * ("max_slots n0 np total_nodes") is what it "finds". */
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct {
  uint32_t x, y, z;
} dim3;

static int device, last_error;
static FILE* out;
static dim3 cfg_grid, cfg_block;
static size_t cfg_shmem;
static struct {
  const void* host;
  const char* name;
} kernels[512];
static int n_kernels;

void** __hipRegisterFatBinary(const void* data) {
  static void* handle;
  (void)data;
  return &handle;
}
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterVar(void** m, void* v, char* h, char* d, int e, size_t s, int c, int g) {
  (void)m, (void)v, (void)h, (void)d, (void)e, (void)s, (void)c, (void)g;
}
void __hipRegisterFunction(void** m, const void* host, char* dev, const char* name, unsigned t, void* a, void* b,
                           void* c, void* d, int* w) {
  (void)m, (void)dev, (void)t, (void)a, (void)b, (void)c, (void)d, (void)w;
  if (n_kernels < 512) {
    kernels[n_kernels].host = host;
    kernels[n_kernels++].name = strdup(name);
  }
}
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t shmem, void* s) {
  (void)s;
  cfg_grid = g;
  cfg_block = b;
  cfg_shmem = shmem;
  return 0;
}
int __hipPopCallConfiguration(dim3* g, dim3* b, size_t* shmem, void** s) {
  *g = cfg_grid;
  *b = cfg_block;
  *shmem = cfg_shmem;
  *s = 0;
  return 0;
}

int hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t shmem, void* s) {
  const char* name = "?";
  (void)shmem, (void)s;
  for (int i = 0; i < n_kernels; ++i)
    if (kernels[i].host == f) name = kernels[i].name;
  if (!out) out = fopen(getenv("HIP_STUB_LOG"), "w");
  fprintf(out, "%s %u %u %u %u %d\n", name, g.x, g.y, g.z, b.x, device);
  fflush(out);
  if (((uint64_t)g.x * b.x >> 32) || ((uint64_t)g.y * b.y >> 32) || g.x == 0 || g.y == 0 || b.x > 1024)
    return last_error = 9; /* hipErrorInvalidConfiguration */
  const char* found = getenv("HIP_STUB_LINEAGE");
  if (found && strstr(name, "k_lineageI")) {
    int32_t* sum = *(int32_t**)args[9];
    sscanf(found, "%d %d %d %d", &sum[0], &sum[1], &sum[2], &sum[3]);
  }
  return 0;
}
int hipGetLastError(void) {
  const int e = last_error;
  last_error = 0;
  return e;
}
const char* hipGetErrorString(int e) { return e == 9 ? "invalid configuration argument" : "no error"; }

int hipGetDevice(int* d) {
  *d = device;
  return 0;
}
int hipSetDevice(int d) {
  device = d;
  return 0;
}
int hipGetSymbolAddress(void** p, const void* sym) {
  (void)sym;
  *p = (void*)(uintptr_t)0x7000000000ull;
  return 0;
}
int hipHostMalloc(void** p, size_t n, unsigned flags) {
  (void)flags;
  *p = calloc(1, n);
  return *p ? 0 : 2;
}
int hipHostFree(void* p) {
  free(p);
  return 0;
}
int hipMemcpy(void* d, const void* s, size_t n, int k) {
  (void)d, (void)s, (void)n, (void)k;
  return 0;
}
int hipMemcpyAsync(void* d, const void* s, size_t n, int k, void* st) {
  (void)d, (void)s, (void)n, (void)k, (void)st;
  return 0;
}
int hipMemsetAsync(void* d, int v, size_t n, void* st) {
  (void)d, (void)v, (void)n, (void)st;
  return 0;
}
int hipStreamCreateWithFlags(void** s, unsigned f) {
  (void)f;
  *s = (void*)1;
  return 0;
}
int hipStreamDestroy(void* s) { (void)s; return 0; }
int hipStreamSynchronize(void* s) { (void)s; return 0; }
int hipStreamBeginCapture(void* s, int m) { (void)s, (void)m; return 0; }
int hipStreamEndCapture(void* s, void** g) {
  (void)s;
  *g = (void*)1;
  return 0;
}
int hipGraphInstantiate(void** e, void* g, void* n, char* l, size_t sz) {
  (void)g, (void)n, (void)l, (void)sz;
  *e = (void*)1;
  return 0;
}
int hipGraphLaunch(void* e, void* s) { (void)e, (void)s; return 0; }
int hipGraphDestroy(void* g) { (void)g; return 0; }
int hipGraphExecDestroy(void* e) { (void)e; return 0; }
int hipEventCreate(void** e) {
  *e = (void*)1;
  return 0;
}
int hipEventDestroy(void* e) { (void)e; return 0; }
int hipEventRecord(void* e, void* s) { (void)e, (void)s; return 0; }
int hipEventSynchronize(void* e) { (void)e; return 0; }
int hipEventElapsedTime(float* t, void* a, void* b) {
  (void)a, (void)b;
  *t = 1;
  return 0;
}
