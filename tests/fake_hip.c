/* The HIP runtime calls libkperf.so makes, answered without a device: launches are written down instead of
 * executed.  Loaded ahead of libkperf.so with global symbols, so that the library binds to these. */
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3;

static int g_dev = 0, g_cus = 256, g_per_cu = 1;
static struct { const void* fn; char name[192]; } g_fn[512];
static int g_n_fn = 0;
static struct { const void* fn; uint32_t grid, block; size_t lds; } g_launch[64];
static int g_n_launch = 0;
static dim3 g_cfg_grid, g_cfg_block;
static size_t g_cfg_lds;
static void* g_cfg_stream;

void fake_device(int dev, int cus, int per_cu) { g_dev = dev; g_cus = cus; g_per_cu = per_cu; }
void fake_forget(void) { g_n_launch = 0; }
int fake_launches(void) { return g_n_launch; }
const char* fake_launch(int i, uint32_t* grid, uint32_t* block, uint64_t* lds) {
  *grid = g_launch[i].grid; *block = g_launch[i].block; *lds = g_launch[i].lds;
  for (int k = 0; k < g_n_fn; ++k)
    if (g_fn[k].fn == g_launch[i].fn) return g_fn[k].name;
  return "?";
}

void** __hipRegisterFatBinary(const void* data) { static void* h; (void)data; return &h; }
void __hipUnregisterFatBinary(void** h) { (void)h; }
void __hipRegisterFunction(void** h, const void* fn, char* device, const char* name, unsigned limit, void* tid, void* bid, dim3* bd,
                           dim3* gd, int* ws) {
  (void)h; (void)device; (void)limit; (void)tid; (void)bid; (void)bd; (void)gd; (void)ws;
  if (g_n_fn < 512) { g_fn[g_n_fn].fn = fn; snprintf(g_fn[g_n_fn++].name, sizeof g_fn[0].name, "%s", name); }
}
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void* stream) {
  g_cfg_grid = grid; g_cfg_block = block; g_cfg_lds = lds; g_cfg_stream = stream;
  return 0;
}
int __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, void** stream) {
  *grid = g_cfg_grid; *block = g_cfg_block; *lds = g_cfg_lds; *stream = g_cfg_stream;
  return 0;
}
int hipLaunchKernel(const void* fn, dim3 grid, dim3 block, void** args, size_t lds, void* stream) {
  (void)args; (void)stream;
  if (g_n_launch < 64) {
    g_launch[g_n_launch].fn = fn; g_launch[g_n_launch].grid = grid.x;
    g_launch[g_n_launch].block = block.x; g_launch[g_n_launch++].lds = lds;
  }
  return 0;
}
int hipGetDevice(int* dev) { *dev = g_dev; return 0; }
int hipDeviceGetAttribute(int* v, int attr, int dev) { (void)attr; (void)dev; *v = g_cus; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* fn, int block, size_t lds) {
  (void)fn; (void)block; (void)lds; *n = g_per_cu; return 0;
}
int hipFuncSetAttribute(const void* fn, int attr, int v) { (void)fn; (void)attr; (void)v; return 0; }
int hipGetLastError(void) { return 0; }
const char* hipGetErrorString(int e) { (void)e; return "no error"; }
int hipEventRecord(void* e, void* s) { (void)e; (void)s; return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int kind, void* stream) {
  (void)d; (void)s; (void)n; (void)kind; (void)stream;
  return 1; /* (no device memory to copy from) */
}
int hipStreamSynchronize(void* s) { (void)s; return 0; }
