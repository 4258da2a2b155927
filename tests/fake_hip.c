/* A HIP runtime without a GPU, for tests of what the library's host side asks of it: memory up to a budget, copies of tables, and a list of the
 * launches with their grids and kernels' names.  Loaded with RTLD_GLOBAL before the library, whose calls then resolve to this file. */
#define _GNU_SOURCE
#include <dlfcn.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;
enum { OK = 0, OOM = 2, BAD_LAUNCH = 9 };

#define SLOTS 512
static struct { void *p; size_t size; } held[SLOTS];
static size_t budget = (size_t)1 << 62, used;
static int last, launches;
static dim3_t grids[64], blocks[64], next_grid, next_block;
static const void *kernels[64];
static size_t next_lds;
static void *next_stream;

void fake_budget(size_t bytes) { budget = bytes; }
size_t fake_used(void) { return used; }
int fake_launches(void) { const int n = launches; launches = 0; return n; }
void fake_launch(int i, uint32_t *out) { memcpy(out, &grids[i], 12); memcpy(out + 3, &blocks[i], 12); }

const char *fake_kernel(int i) { Dl_info d; return dladdr(kernels[i], &d) && d.dli_sname ? d.dli_sname : ""; }

int hipMalloc(void **p, size_t size) {
  for (int i = 0; i < SLOTS; ++i)
    if (!held[i].p) {
      if (used + size > budget) return last = OOM;
      held[i].p = *p = calloc(1, size < ((size_t)64 << 20) ? size + 1 : 256);   /* (what is larger is never touched here) */
      held[i].size = size;
      used += size;
      return OK;
    }
  abort();
}
int hipFree(void *p) {
  for (int i = 0; i < SLOTS; ++i)
    if (held[i].p == p) { used -= held[i].size; held[i].p = NULL; free(p); return OK; }
  abort();                                                  /* not ours, or freed before */
}
int hipMemcpy(void *to, const void *from, size_t n, int kind) { (void)kind; memcpy(to, from, n); return OK; }
int hipGetDeviceCount(int *n) { *n = 1; return OK; }
int hipSetDevice(int d) { return d; }
int hipDeviceSynchronize(void) { return OK; }
int hipDeviceGetAttribute(int *v, int which, int d) {
  (void)d;
  *v = which == LDS_ATTRIBUTE ? 163840 : which == CU_ATTRIBUTE ? 256 : -1;
  return *v < 0;
}
int hipFuncSetAttribute(const void *f, int which, int v) { (void)f; (void)which; return v > 163840; }
static char symbol[1];
int hipGetSymbolAddress(void **p, const void *s) { (void)s; *p = symbol; return OK; }
int hipGetLastError(void) { const int e = last; last = OK; return e; }
const char *hipGetErrorString(int e) { return e == OOM ? "out of memory" : "launch refused"; }
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t lds, void *stream) { next_grid = g; next_block = b; next_lds = lds; next_stream = stream; return OK; }
int __hipPopCallConfiguration(dim3_t *g, dim3_t *b, size_t *lds, void **stream) { *g = next_grid; *b = next_block; *lds = next_lds; *stream = next_stream; return OK; }
int hipLaunchKernel(const void *f, dim3_t g, dim3_t b, void **args, size_t lds, void *stream) {
  (void)args; (void)lds; (void)stream;
  if ((uint64_t)g.x * b.x >> 32 || (uint64_t)g.y * b.y >> 32) return last = BAD_LAUNCH;
  if (launches < 64) { grids[launches] = g; blocks[launches] = b; kernels[launches] = f; }
  ++launches;
  return OK;
}
