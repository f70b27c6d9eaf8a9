/* Stand-ins for the HIP runtime calls libdvbm.so makes, which record themselves: loaded into the global scope before the
 * library, they let its host code run without a GPU.  Buffers are host addresses that nothing dereferences, except the
 * four extrema dvbm_init copies back. */
#define _GNU_SOURCE
#include <dlfcn.h>
#include <stdarg.h>
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3;

static char log_text[1 << 20];
static size_t log_len;
static struct { char text[64]; int count; } workgroups[8];  /* per compute unit, by a part of the kernel's name; else 1 */
static int n_workgroups;
static dim3 pushed_grid, pushed_block;
static size_t pushed_shared;
static void* pushed_stream;

static void record(const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  log_len += (size_t)vsnprintf(log_text + log_len, sizeof(log_text) - log_len, fmt, ap);
  va_end(ap);
  if (log_len >= sizeof(log_text)) abort();
}

const char* recorder_log(void) { return log_text; }
void recorder_clear(void) { log_text[log_len = 0] = 0; }
void recorder_forget_workgroups(void) { n_workgroups = 0; }
void recorder_set_workgroups(const char* text, int count) {
  if (n_workgroups == 8) abort();
  snprintf(workgroups[n_workgroups].text, sizeof(workgroups[0].text), "%s", text);
  workgroups[n_workgroups++].count = count;
}

static const char* kernel_name(const void* kernel) {
  Dl_info info;
  return dladdr(kernel, &info) && info.dli_sname ? info.dli_sname : "?";
}

int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, void* stream) {
  pushed_grid = grid;
  pushed_block = block;
  pushed_shared = shared;
  pushed_stream = stream;
  return 0;
}
int __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, void** stream) {
  *grid = pushed_grid;
  *block = pushed_block;
  *shared = pushed_shared;
  *stream = pushed_stream;
  return 0;
}
int hipLaunchKernel(const void* kernel, dim3 grid, dim3 block, void** args, size_t shared, void* stream) {
  (void)args, (void)shared, (void)stream;
  record("launch %s %u %u\n", kernel_name(kernel), grid.x * grid.y * grid.z, block.x * block.y * block.z);
  return 0;
}
int hipGetLastError(void) { return 0; }
const char* hipGetErrorString(int e) { (void)e; return "recorded"; }
int hipStreamSynchronize(void* s) { (void)s; record("hipStreamSynchronize\n"); return 0; }
int hipMemcpyAsync(void* dst, const void* src, size_t n, int kind, void* s) {
  static const double extrema[4] = {1.0, 1.0, -1.0, -1.0};
  (void)src, (void)s;
  record("hipMemcpyAsync\n");
  if (kind == 2) memcpy(dst, extrema, n < sizeof(extrema) ? n : sizeof(extrema));
  return 0;
}
int hipMemsetAsync(void* p, int v, size_t n, void* s) { (void)p, (void)v, (void)n, (void)s; record("hipMemsetAsync\n"); return 0; }
int hipGetSymbolAddress(void** p, const void* sym) { (void)sym; record("hipGetSymbolAddress\n"); *p = (void*)(uintptr_t)4096; return 0; }
int hipGetDevice(int* d) { record("hipGetDevice\n"); *d = 0; return 0; }
int hipDeviceGetAttribute(int* v, int attr, int d) { (void)attr, (void)d; record("hipDeviceGetAttribute\n"); *v = 256; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int block, size_t shared) {
  (void)block, (void)shared;
  record("hipOccupancyMaxActiveBlocksPerMultiprocessor\n");
  *n = 1;
  for (int k = 0; k < n_workgroups; ++k)
    if (strstr(kernel_name(f), workgroups[k].text)) *n = workgroups[k].count;
  return 0;
}
