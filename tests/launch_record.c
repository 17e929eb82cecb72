/* Stands in for the HIP runtime in a process without a GPU: kernels are registered by name, a launch is noted
 * instead of run, and a grid the runtime refuses (2^32 or more threads along x) is refused.  Loaded globally ahead of libdll_conv.so, so that the library's calls land here. */
#include <stddef.h>
#include <stdio.h>
#include <string.h>

typedef struct { unsigned x, y, z; } dim3;
enum { kMaxKernels = 1024, kMaxLaunches = 256 };
static struct { const void *handle; const char *name; } kernels[kMaxKernels];
static int n_kernels, n_launches, last_error;
static struct { const char *name; dim3 grid, block; } launches[kMaxLaunches];
static struct { dim3 grid, block; size_t lds; void *stream; } pending;

void **__hipRegisterFatBinary(const void *data) { static void *h; (void)data; return &h; }
void __hipUnregisterFatBinary(void **h) { (void)h; }
void __hipRegisterFunction(void **m, const void *handle, char *device, const char *name, unsigned l, void *t, void *b, void *bd, void *gd, int *w) {
  (void)m; (void)device; (void)l; (void)t; (void)b; (void)bd; (void)gd; (void)w;
  if (n_kernels < kMaxKernels && strstr(name, "dllk")) { kernels[n_kernels].handle = handle; kernels[n_kernels++].name = name; }
}
void __hipRegisterVar(void **m, void *v, char *h, char *d, int e, size_t s, int c, int g) { (void)m; (void)v; (void)h; (void)d; (void)e; (void)s; (void)c; (void)g; }
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void *stream) {
  pending.grid = grid; pending.block = block; pending.lds = lds; pending.stream = stream;
  return 0;
}
int __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, void **stream) {
  *grid = pending.grid; *block = pending.block; *lds = pending.lds; *stream = pending.stream;
  return 0;
}
int hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t lds, void *stream) {
  const char *name = "?";
  (void)args; (void)lds; (void)stream;
  for (int i = 0; i < n_kernels; ++i)
    if (kernels[i].handle == f) name = kernels[i].name;
  if (!grid.x || !grid.y || !grid.z || (unsigned long)grid.x * block.x >= 1ul << 32) return last_error = 9;
  if (n_launches < kMaxLaunches) { launches[n_launches].name = name; launches[n_launches].grid = grid; launches[n_launches++].block = block; }
  return 0;
}
int hipGetLastError(void) { const int e = last_error; last_error = 0; return e; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int *v, int a, int d) { (void)v; (void)a; (void)d; return 1; }   /* the library's own figures stand in */
int hipFuncSetAttribute(const void *f, int a, int v) { (void)f; (void)a; (void)v; return 0; }

/* The launches since the last call, one a line: name, grid, block. */
void take_launches(char *out, size_t room) {
  size_t at = 0;
  out[0] = 0;
  for (int i = 0; i < n_launches && at + 512 < room; ++i)
    at += (size_t)snprintf(out + at, room - at, "%.400s %u %u %u %u\n", launches[i].name, launches[i].grid.x, launches[i].grid.y, launches[i].grid.z, launches[i].block.x);
  n_launches = 0;
}
