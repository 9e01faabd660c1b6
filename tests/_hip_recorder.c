/* A HIP runtime that runs nothing: it hands out host memory, notes the name and grid of every kernel
 * launched, and refuses allocations above a limit.  Loaded before the library (RTLD_GLOBAL), it shows on
 * the CPU which kernels a call enqueues and what a refused allocation does.  Untouched memory is zero, so
 * a solve that waits for its count of open right-hand sides reads that none is left. */
#define _GNU_SOURCE
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3;
typedef int err_t;

enum { MAXK = 4096, MAXL = 65536 };
static struct { const void* host; const char* name; } kern[MAXK];
static int nkern;
static struct { const char* name; dim3 grid, block; } launch[MAXL];
static int nlaunch;
static size_t limit = (size_t)-1, largest;
static int capturing;

void rec_reset(void) { nlaunch = 0; }
int rec_count(void) { return nlaunch; }
const char* rec_name(int i) { return launch[i].name; }
long rec_threads(int i) { return (long)launch[i].block.x * launch[i].block.y; }
long rec_blocks(int i) { return (long)launch[i].grid.x * launch[i].grid.y; }
void rec_limit(size_t n) { limit = n; largest = 0; }
size_t rec_largest(void) { return largest; }
void rec_capturing(int on) { capturing = on; }

static err_t give(void** p, size_t n) {
  if (n > largest) largest = n;
  *p = NULL;
  if (n > limit) return 2; /* hipErrorOutOfMemory */
  *p = calloc(1, n ? n : 1);
  return *p ? 0 : 2;
}

void** __hipRegisterFatBinary(const void* d) { static void* h; (void)d; return &h; }
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterFunction(void** m, const void* host, char* dev, const char* name, unsigned lim, void* a, void* b,
                           void* c, void* d, int* w) {
  (void)m; (void)dev; (void)lim; (void)a; (void)b; (void)c; (void)d; (void)w;
  if (nkern < MAXK) { kern[nkern].host = host; kern[nkern++].name = name; }
}
void __hipRegisterVar(void** m, void* v, char* h, char* d, int e, size_t n, int c, int g) {
  (void)m; (void)v; (void)h; (void)d; (void)e; (void)n; (void)c; (void)g;
}
static struct { dim3 grid, block; size_t lds; void* s; } cfg;
err_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, void* s) {
  cfg.grid = g; cfg.block = b; cfg.lds = lds; cfg.s = s;
  return 0;
}
err_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, void** s) {
  *g = cfg.grid; *b = cfg.block; *lds = cfg.lds; *s = cfg.s;
  return 0;
}
err_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t lds, void* s) {
  (void)args; (void)lds; (void)s;
  const char* name = "?";
  for (int i = 0; i < nkern; ++i)
    if (kern[i].host == f) name = kern[i].name;
  if (nlaunch < MAXL) { launch[nlaunch].name = name; launch[nlaunch].grid = g; launch[nlaunch++].block = b; }
  return 0;
}
err_t hipLaunchCooperativeKernel(const void* f, dim3 g, dim3 b, void** args, unsigned lds, void* s) {
  return hipLaunchKernel(f, g, b, args, lds, s);
}

err_t hipMalloc(void** p, size_t n) { return give(p, n); }
err_t hipHostMalloc(void** p, size_t n, unsigned f) { (void)f; return give(p, n); }
err_t hipFree(void* p) { free(p); return 0; }
err_t hipHostFree(void* p) { free(p); return 0; }
err_t hipHostGetDevicePointer(void** d, void* h, unsigned f) { (void)f; *d = h; return 0; }
err_t hipGetSymbolAddress(void** p, const void* s) { static double a[1 << 16]; (void)s; *p = a; return 0; }
err_t hipMemcpy(void* d, const void* s, size_t n, int k) { (void)k; memcpy(d, s, n); return 0; }
err_t hipMemcpyAsync(void* d, const void* s, size_t n, int k, void* st) { (void)st; return hipMemcpy(d, s, n, k); }
err_t hipMemset(void* d, int v, size_t n) { memset(d, v, n); return 0; }
err_t hipMemsetAsync(void* d, int v, size_t n, void* s) { (void)s; return hipMemset(d, v, n); }
err_t hipGetDevice(int* d) { *d = 0; return 0; }
err_t hipDeviceGetAttribute(int* v, int a, int d) { (void)a; (void)d; *v = 256; return 0; }
err_t hipGetDevicePropertiesR0600(void* p, int d) { /* 256 compute units, 256 everything */
  (void)d;
  for (int i = 0; i < 64; ++i) ((int*)p)[64 + i] = 256;
  return 0;
}
err_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int b, size_t l) {
  (void)f; (void)l; *n = b > 512 ? 1 : 2; return 0;
}
err_t hipFuncSetAttribute(const void* f, int a, int v) { (void)f; (void)a; (void)v; return 0; }
err_t hipDeviceSynchronize(void) { return 0; }
err_t hipStreamSynchronize(void* s) { (void)s; return 0; }
err_t hipStreamCreateWithFlags(void** s, unsigned f) { (void)f; *s = (void*)1; return 0; }
err_t hipStreamDestroy(void* s) { (void)s; return 0; }
err_t hipStreamIsCapturing(void* s, int* st) { (void)s; *st = capturing; return 0; }
err_t hipStreamBeginCapture(void* s, int m) { (void)s; (void)m; return 0; }
err_t hipStreamEndCapture(void* s, void** g) { (void)s; *g = (void*)1; return 0; }
err_t hipGraphInstantiate(void** e, void* g, void* n, char* b, size_t z) { (void)g; (void)n; (void)b; (void)z; *e = (void*)1; return 0; }
err_t hipGraphLaunch(void* e, void* s) { (void)e; (void)s; return 0; }
err_t hipGraphDestroy(void* g) { (void)g; return 0; }
err_t hipGraphExecDestroy(void* g) { (void)g; return 0; }
err_t hipEventCreate(void** e) { *e = (void*)1; return 0; }
err_t hipEventCreateWithFlags(void** e, unsigned f) { (void)f; *e = (void*)1; return 0; }
err_t hipEventDestroy(void* e) { (void)e; return 0; }
err_t hipEventRecord(void* e, void* s) { (void)e; (void)s; return 0; }
err_t hipEventSynchronize(void* e) { (void)e; return 0; }
err_t hipEventElapsedTime(float* t, void* a, void* b) { (void)a; (void)b; *t = 1.0f; return 0; }
const char* hipGetErrorString(err_t e) { return e == 2 ? "out of memory" : "error"; }
err_t hipGetLastError(void) { return 0; }
