/* A stand-in for the HIP runtime, for tests of the library's host side on
 * machines without a GPU: it launches nothing and logs every kernel launch and
 * copy.  Loaded with RTLD_GLOBAL before the library, its definitions are taken
 * for the library's runtime calls.  fake_alloc declares a piece of memory. */
#include <stdarg.h>
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3;
enum { kInvalidValue = 1 };

static char logged[1 << 20];
static size_t used;
static void note(const char* fmt, ...) {
  va_list a;
  va_start(a, fmt);
  int n = vsnprintf(logged + used, sizeof(logged) - used, fmt, a);
  va_end(a);
  if (n > 0 && used + n < sizeof(logged)) used += n;
}
const char* fake_log(void) { return logged; }
void fake_clear(void) { used = 0; logged[0] = 0; }

static struct { uintptr_t base; size_t size; int type, device; } mem[64];
static int nmem;
void fake_alloc(uintptr_t base, size_t size, int type, int device) {
  mem[nmem].base = base;
  mem[nmem].size = size;
  mem[nmem].type = type;
  mem[nmem++].device = device;
}
static int find(const void* p) {
  for (int j = 0; j < nmem; ++j)
    if ((uintptr_t)p - mem[j].base < mem[j].size) return j;
  return -1;
}
static int reaches_past(const void* p, size_t n) {
  const int j = find(p);
  return j >= 0 && (uintptr_t)p - mem[j].base + n > mem[j].size;
}

static const void* fun[4096];
static const char* fun_name[4096];
static int nfun;
void** __hipRegisterFatBinary(const void* d) { static void* h; (void)d; return &h; }
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterFunction(void** m, const void* host, char* dev, const char* name, unsigned limit,
                           void* t, void* b, dim3* bd, dim3* gd, int* w) {
  (void)m, (void)dev, (void)limit, (void)t, (void)b, (void)bd, (void)gd, (void)w;
  fun[nfun] = host;
  fun_name[nfun++] = name;
}
void __hipRegisterVar(void** m, void* var, char* host, char* dev, int ext, size_t size, int c, int g) {
  (void)m, (void)var, (void)host, (void)dev, (void)ext, (void)size, (void)c, (void)g;
}
static dim3 cfg_grid, cfg_block;
static size_t cfg_shared;
static void* cfg_stream;
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, void* st) {
  cfg_grid = g, cfg_block = b, cfg_shared = s, cfg_stream = st;
  return 0;
}
int __hipPopCallConfiguration(dim3* g, dim3* b, size_t* s, void** st) {
  *g = cfg_grid, *b = cfg_block, *s = cfg_shared, *st = cfg_stream;
  return 0;
}
int hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t shared, void* st) {
  (void)shared, (void)st;
  const char* name = "?";
  for (int j = 0; j < nfun; ++j)
    if (fun[j] == f) name = fun_name[j];
  /* the z-marching kernels' last argument: the planes of a chunk */
  const int zc = strstr(name, "fused3d") ? *(const int*)args[6] : 0;
  note("launch %s %u %u %u %u %u %u %d\n", name, g.x, g.y, g.z, b.x, b.y, b.z, zc);
  return 0;
}
int hipMemcpyAsync(void* dst, const void* src, size_t n, int kind, void* st) {
  (void)kind, (void)st;
  if (reaches_past(dst, n) || reaches_past(src, n)) return kInvalidValue;
  note("copy %zu\n", n);
  return 0;
}
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipSetDevice(int d) { (void)d; return 0; }
int hipGetLastError(void) { return 0; }
const char* hipGetErrorString(int e) { return e ? "invalid argument" : "no error"; }
int hipGetSymbolAddress(void** p, const void* s) { *p = (void*)(uintptr_t)0x1000; (void)s; return 0; }
int hipStreamSynchronize(void* s) { (void)s; return 0; }
int hipDeviceGetAttribute(int* v, int a, int d) { (void)a, (void)d; *v = 256; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int t, size_t s) {
  (void)f, (void)t, (void)s;
  *n = 1;
  return 0;
}
/* type, device, device and host pointer, managed, flags */
struct attributes { int type, device; void *dev, *host; int managed; unsigned flags; };
int hipPointerGetAttributes(struct attributes* a, const void* p) {
  const int j = find(p);
  if (j < 0) return kInvalidValue;
  memset(a, 0, sizeof(*a));
  a->type = mem[j].type;
  a->device = mem[j].device;
  return 0;
}
int hipMemGetAddressRange(void** base, size_t* size, void* p) {
  const int j = find(p);
  if (j < 0) return kInvalidValue;
  *base = (void*)mem[j].base;
  *size = mem[j].size;
  return 0;
}
