/* The HIP functions that libgnmr.so calls, on host memory: no kernel runs, launches
 * are counted, and any call can be made to fail.  Linked into a test program, they
 * take the place of the HIP runtime's. */
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3;

int fake_launches;       /* kernels launched since it was last cleared */
int fake_fail_launches;  /* that many launches from now fail */
int fake_fail_events;    /* that many event records from now fail */
static int last_error;   /* of a launch */

static int fails(int* left) { return *left > 0 ? --*left, 719 : 0; }

void** __hipRegisterFatBinary(const void* data) { return (void**)data; }
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterFunction(void** m, const void* f, char* d, const char* n, unsigned lim, void* a,
                           void* b, void* c, void* e, int* w) {
  (void)m, (void)f, (void)d, (void)n, (void)lim, (void)a, (void)b, (void)c, (void)e, (void)w;
}
void __hipRegisterVar(void** m, void* v, char* h, char* d, int ext, size_t size, int c, int g) {
  (void)m, (void)v, (void)h, (void)d, (void)ext, (void)size, (void)c, (void)g;
}

static dim3 cfg_grid, cfg_block;
static size_t cfg_lds;
static void* cfg_stream;
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void* stream) {
  cfg_grid = grid, cfg_block = block, cfg_lds = lds, cfg_stream = stream;
  return 0;
}
int __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, void** stream) {
  *grid = cfg_grid, *block = cfg_block, *lds = cfg_lds, *stream = cfg_stream;
  return 0;
}
int hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t lds, void* stream) {
  (void)f, (void)args, (void)lds, (void)stream;
  if (fake_fail_launches > 0) return last_error = fails(&fake_fail_launches);
  if (!grid.x || !block.x || (uint64_t)grid.x * block.x > UINT32_MAX || block.x > 1024)
    return last_error = 9;
  ++fake_launches;
  return 0;
}
int hipGetLastError(void) {
  const int e = last_error;
  last_error = 0;
  return e;
}
const char* hipGetErrorString(int e) { return e ? "made to fail" : "no error"; }

int hipGetDevice(int* d) { return *d = 0; }
int hipSetDevice(int d) { return d != 0; }
int hipDeviceSynchronize(void) { return 0; }
int hipStreamSynchronize(void* s) { return (void)s, 0; }
int hipMalloc(void** p, size_t n) { return (*p = malloc(n ? n : 1)) == NULL; }
int hipFree(void* p) { return free(p), 0; }
int hipHostMalloc(void** p, size_t n, unsigned flags) { return (void)flags, hipMalloc(p, n); }
int hipHostFree(void* p) { return hipFree(p); }
int hipMemcpy(void* to, const void* from, size_t n, int kind) {
  return (void)kind, memcpy(to, from, n), 0;
}
int hipMemcpyAsync(void* to, const void* from, size_t n, int kind, void* s) {
  return (void)s, hipMemcpy(to, from, n, kind);
}
int hipMemsetAsync(void* p, int v, size_t n, void* s) { return (void)s, memset(p, v, n), 0; }
int hipGetSymbolAddress(void** p, const void* s) { return (void)s, *p = NULL, 1; }

int hipEventCreate(void** e) { return hipMalloc(e, 1); }
int hipEventCreateWithFlags(void** e, unsigned flags) { return (void)flags, hipMalloc(e, 1); }
int hipEventDestroy(void* e) { return hipFree(e); }
int hipEventRecord(void* e, void* s) { return (void)e, (void)s, fails(&fake_fail_events); }
int hipEventSynchronize(void* e) { return (void)e, 0; }
int hipEventElapsedTime(float* ms, void* a, void* b) { return (void)a, (void)b, *ms = 0, 0; }
