/* The HIP runtime calls libkperf.so makes, answered without a device: launches are written down instead of
 * executed.  Loaded ahead of libkperf.so with global symbols, so that the library binds to these.
 * Host memory that kernels can write is real memory here, in allocations that fake_reset() takes back, and the kernel that
 * writes a trace's header to it is carried out, unless fake_silent() says otherwise. */
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
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
/* the header of the trace at any device address, and what became of the reads */
static uint32_t g_header[16];
static int g_silent = 0, g_header_kernels = 0, g_header_copies = 0;
static struct { char* at; size_t size; uint64_t id; } g_host[64];
static int g_n_host = 0, g_host_frees = 0, g_stray_writes = 0, g_unguarded = 0;
static uint64_t g_next_id = 1;
static _Thread_local int g_capture_mode = 0; /* global; 2: relaxed */
void fake_header(const uint32_t* words) { memcpy(g_header, words, sizeof g_header); }
void fake_silent(int on) { g_silent = on; }
void fake_reset(void) { g_n_host = 0; } /* (the memory itself stays, so that a write to it can be seen) */
int fake_count(int which) {
  const int v[] = {g_header_kernels, g_header_copies, g_n_host, g_host_frees, g_stray_writes, g_unguarded};
  return v[which];
}
static int host_block(const void* p) {
  for (int i = 0; i < g_n_host; ++i)
    if ((const char*)p >= g_host[i].at && (const char*)p < g_host[i].at + g_host[i].size) return i;
  return -1;
}
int hipHostMalloc(void** p, size_t n, unsigned flags) {
  (void)flags;
  g_unguarded += g_capture_mode != 2;
  if (g_n_host == 64) return 2;
  *p = calloc(1, n);
  g_host[g_n_host].at = *p; g_host[g_n_host].size = n; g_host[g_n_host++].id = g_next_id++;
  return 0;
}
int hipHostFree(void* p) {
  (void)p;
  g_unguarded += g_capture_mode != 2;
  ++g_host_frees;
  return 0;
}
int hipThreadExchangeStreamCaptureMode(int* mode) { const int m = g_capture_mode; g_capture_mode = *mode; *mode = m; return 0; }
int hipStreamIsCapturing(void* s, int* status) { (void)s; *status = 0; return 0; }
int hipPointerGetAttributes(int* at, const void* p) { (void)p; at[0] = 2; at[1] = g_dev; return 0; } /* device memory */
int hipPointerGetAttribute(void* data, int which, void* p) {
  const int i = host_block(p);
  if (which != 7 || i < 0) return 1;
  *(uint64_t*)data = g_host[i].id;
  return 0;
}
int hipMemGetAddressRange(void** base, size_t* size, void* p) { *base = p; *size = (size_t)1 << 30; return 0; }

int hipLaunchKernel(const void* fn, dim3 grid, dim3 block, void** args, size_t lds, void* stream) {
  (void)stream;
  for (int k = 0; k < g_n_fn; ++k) {
    if (g_fn[k].fn != fn || !strstr(g_fn[k].name, "kp_header_to_host")) continue;
    uint32_t* to = *(uint32_t**)args[1];
    __atomic_fetch_add(&g_header_kernels, 1, __ATOMIC_RELAXED);
    if (host_block(to) < 0) { __atomic_fetch_add(&g_stray_writes, 1, __ATOMIC_RELAXED); return 0; }
    if (g_silent) return 0;
    memcpy(to, g_header, sizeof g_header);
    __atomic_store_n(to + 16, *(uint32_t*)args[2], __ATOMIC_RELEASE);
    return 0;
  }
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
  (void)s; (void)kind; (void)stream;
  if (!g_header[0] || n != sizeof g_header) return 1; /* (no device memory to copy from) */
  memcpy(d, g_header, n);
  __atomic_fetch_add(&g_header_copies, 1, __ATOMIC_RELAXED);
  return 0;
}
int hipStreamSynchronize(void* s) { (void)s; return 0; }
