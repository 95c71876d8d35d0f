/* The few entry points of the HIP runtime that the library uses, over host memory: copies are memcpy, a kernel launch is an
 * entry in a list.  With it the library's host side (what it launches, with which operands, in what order, and what it does when
 * a launch fails) runs on a CPU.  Loaded into a process of its own before the library. */
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

typedef struct {
  uint32_t x, y, z;
} grid_t;
typedef struct {
  const char *name;
  grid_t grid;
  uint8_t args[256]; /* the first bytes of the LayerNorm parameter reduce's only argument */
} launch_t;

static const void **fn;
static const char **fn_name;
static size_t n_fn, cap_fn;
static launch_t *list;
static size_t n_list, cap_list;
static int64_t fail_at = -1; /* launches until one fails (negative: never) */
static int last;

size_t host_launches(void) { return n_list; }
const launch_t *host_launch(size_t i) { return &list[i]; }
void host_clear(int64_t fail_in) { n_list = 0, fail_at = fail_in, last = 0; }

void **__hipRegisterFatBinary(const void *data) {
  static void *h;
  (void)data;
  return &h;
}
void __hipUnregisterFatBinary(void **h) { (void)h; }
void __hipRegisterVar(void) {}
void __hipRegisterFunction(void **h, const void *f, char *dev, const char *name) {
  (void)h, (void)dev;
  if (n_fn == cap_fn) {
    cap_fn = cap_fn ? 2 * cap_fn : 1024;
    fn = realloc(fn, cap_fn * sizeof *fn);
    fn_name = realloc(fn_name, cap_fn * sizeof *fn_name);
  }
  fn[n_fn] = f;
  fn_name[n_fn++] = name;
}

static struct {
  grid_t grid, block;
  size_t smem;
  void *stream;
} call;
int __hipPushCallConfiguration(grid_t grid, grid_t block, size_t smem, void *stream) {
  call.grid = grid, call.block = block, call.smem = smem, call.stream = stream;
  return 0;
}
int __hipPopCallConfiguration(grid_t *grid, grid_t *block, size_t *smem, void **stream) {
  *grid = call.grid, *block = call.block, *smem = call.smem, *stream = call.stream;
  return 0;
}
int hipLaunchKernel(const void *f, grid_t grid, grid_t block, void **args, size_t smem, void *stream) {
  size_t i;
  (void)smem, (void)stream;
  if (fail_at >= 0 && fail_at-- == 0) return last = 1;
  if ((uint64_t)grid.x * block.x >> 32 || (uint64_t)grid.y * block.y >> 32 || (uint64_t)grid.z * block.z >> 32) return last = 9; /* as the runtime does */
  if (n_list == cap_list) list = realloc(list, (cap_list = cap_list ? 2 * cap_list : 1024) * sizeof *list);
  list[n_list].name = "";
  list[n_list].grid = grid;
  for (i = 0; i < n_fn; ++i)
    if (fn[i] == f) list[n_list].name = fn_name[i];
  if (strstr(list[n_list].name, "ln_param_reduce")) memcpy(list[n_list].args, args[0], sizeof list[n_list].args);
  ++n_list;
  return 0;
}
int hipGetLastError(void) {
  const int e = last;
  last = 0;
  return e;
}
const char *hipGetErrorString(int e) { return e ? "launch refused" : "no error"; }
int hipMemcpy(void *dst, const void *src, size_t n, int kind) {
  (void)kind;
  memcpy(dst, src, n);
  return 0;
}
int hipMemcpyAsync(void *dst, const void *src, size_t n, int kind, void *stream) {
  (void)stream;
  return hipMemcpy(dst, src, n, kind);
}
int hipGetSymbolAddress(void **p, const void *symbol) {
  static uint64_t mem[8192];
  (void)symbol;
  *p = mem;
  return 0;
}
int hipGetDevice(int *d) {
  *d = 0;
  return 0;
}
int hipFuncSetAttribute(const void *f, int attr, int value) {
  (void)f, (void)attr, (void)value;
  return 0;
}
int hipDeviceSynchronize(void) { return 0; }
int hipStreamSynchronize(void *s) {
  (void)s;
  return 0;
}
int hipEventCreate(void **e) {
  *e = &last;
  return 0;
}
int hipEventCreateWithFlags(void **e, unsigned flags) {
  (void)flags;
  return hipEventCreate(e);
}
int hipEventDestroy(void *e) {
  (void)e;
  return 0;
}
int hipEventRecord(void *e, void *s) {
  (void)e, (void)s;
  return 0;
}
int hipEventSynchronize(void *e) {
  (void)e;
  return 0;
}
int hipEventElapsedTime(float *ms, void *a, void *b) {
  (void)a, (void)b;
  *ms = 0.f;
  return 0;
}
