/* A HIP runtime without a device, for host-side tests: the library's launches
 * are recorded instead of run, and a launch that the hardware limits exclude
 * (160 KB of LDS per workgroup, 65536 blocks in y and z, 1024 threads, a
 * 32-bit number of work items in x) is refused with the sticky error that the
 * runtime gives.  Device memory is host memory. */
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;
typedef struct { const char* name; dim3_t grid, block; uint64_t lds; int refused; } launch_t;

enum { kMaxFns = 4096, kMaxLaunches = 65536 };
static struct { const void* host; const char* name; } fns[kMaxFns];
static int n_fns;
static launch_t launches[kMaxLaunches];
static int n_launches, last_error;
static struct { dim3_t grid, block; size_t lds; void* stream; } config;

void** __hipRegisterFatBinary(const void* data) { (void)data; static void* module; return &module; }
void __hipUnregisterFatBinary(void** modules) { (void)modules; }
void __hipRegisterFunction(void** modules, const void* host, char* device, const char* name, unsigned limit, void* tid,
                           void* bid, dim3_t* block, dim3_t* grid, int* wsize) {
  (void)modules, (void)device, (void)limit, (void)tid, (void)bid, (void)block, (void)grid, (void)wsize;
  if (n_fns < kMaxFns) fns[n_fns].host = host, fns[n_fns++].name = name;
}
void __hipRegisterVar(void** modules, void* var, char* host, char* name, int ext, size_t size, int constant, int global) {
  (void)modules, (void)var, (void)host, (void)name, (void)ext, (void)size, (void)constant, (void)global;
}
int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t lds, void* stream) {
  config.grid = grid, config.block = block, config.lds = lds, config.stream = stream;
  return 0;
}
int __hipPopCallConfiguration(dim3_t* grid, dim3_t* block, size_t* lds, void** stream) {
  *grid = config.grid, *block = config.block, *lds = config.lds, *stream = config.stream;
  return 0;
}
int hipLaunchKernel(const void* host, dim3_t grid, dim3_t block, void** args, size_t lds, void* stream) {
  (void)args, (void)stream;
  launch_t l = {"?", grid, block, lds, 0};
  for (int k = 0; k < n_fns; ++k)
    if (fns[k].host == host) l.name = fns[k].name;
  const uint64_t threads = (uint64_t)block.x * block.y * block.z;
  l.refused = lds > 160 * 1024 || grid.y > 65536 || grid.z > 65536 || threads == 0 || threads > 1024 ||
              (uint64_t)grid.x * grid.y * grid.z == 0 || (uint64_t)grid.x * block.x > UINT32_MAX;
  if (n_launches < kMaxLaunches) launches[n_launches++] = l;
  if (l.refused) last_error = 1;
  return l.refused;
}
int hipFuncSetAttribute(const void* host, int attr, int value) {
  (void)host, (void)attr;
  return value > 160 * 1024;
}
int hipGetLastError(void) {
  const int e = last_error;
  last_error = 0;
  return e;
}
int hipGetDevice(int* device) { *device = 0; return 0; }
int hipGetSymbolAddress(void** p, const void* symbol) {
  (void)symbol;
  static char scratch[256];
  *p = scratch;
  return 0;
}
int hipMalloc(void** p, size_t bytes) { return (*p = malloc(bytes)) == NULL; }
int hipFree(void* p) { free(p); return 0; }
int hipMemcpy(void* dst, const void* src, size_t bytes, int kind) { (void)kind; memcpy(dst, src, bytes); return 0; }
int hipEventCreate(void** e) { *e = NULL; return 0; }
int hipEventDestroy(void* e) { (void)e; return 0; }
int hipEventRecord(void* e, void* s) { (void)e, (void)s; return 0; }
int hipEventSynchronize(void* e) { (void)e; return 0; }
int hipEventElapsedTime(float* ms, void* a, void* b) { (void)a, (void)b; *ms = 0; return 0; }

void fake_reset(void) { n_launches = 0, last_error = 0; }
int fake_count(void) { return n_launches; }
void fake_get(int k, const char** name, uint32_t* dims, uint64_t* lds, int* refused) {
  const launch_t* l = &launches[k];
  *name = l->name;
  const uint32_t v[6] = {l->grid.x, l->grid.y, l->grid.z, l->block.x, l->block.y, l->block.z};
  memcpy(dims, v, sizeof v);
  *lds = l->lds, *refused = l->refused;
}
