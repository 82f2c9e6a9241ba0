/* A HIP runtime for the host alone, loaded in front of the real one: device
 * memory is host memory, copies and fills are done at once, and a kernel launch
 * does nothing but report itself.  For tests of what the library's host code
 * asks of the runtime (which kernels, how many allocations and copies, what it
 * does when one fails); the callbacks may be left null. */
#include <stdlib.h>
#include <string.h>

typedef struct { unsigned x, y, z; } dim3;

/* a launch: kernel name, workgroups, argument pointers; nonzero: it fails */
int (*stub_on_launch)(const char *name, unsigned blocks, void **args);
/* a call of the runtime by name; nonzero: it fails (hipErrorUnknown) */
int (*stub_on_call)(const char *name);

static int last_error;
static int call(const char *name) {
  const int e = stub_on_call && stub_on_call(name) ? 999 : 0;
  if (e) last_error = e;
  return e;
}

size_t stub_var_bytes;  /* device variables */
static struct { const void *key; const char *name; void *mem; } table[4096];
static int entries;

void **__hipRegisterFatBinary(const void *d) { static void *m; (void)d; return &m; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterFunction(void **m, const void *host, char *dev, const char *name, unsigned lim, void *tid,
                           void *bid, dim3 *bd, dim3 *gd, int *ws) {
  (void)m; (void)dev; (void)lim; (void)tid; (void)bid; (void)bd; (void)gd; (void)ws;
  if (entries == 4096) abort();
  table[entries].key = host;
  table[entries++].name = name;
}
void __hipRegisterVar(void **m, void *host, char *dev, const char *name, int ext, size_t size, int cst, int gl) {
  (void)m; (void)dev; (void)ext; (void)cst; (void)gl;
  if (entries == 4096) abort();
  table[entries].key = host;
  table[entries].name = name;
  table[entries++].mem = calloc(1, size);
  stub_var_bytes += size;
}

static struct { dim3 g, b; size_t sh; void *st; } conf;
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t sh, void *st) {
  conf.g = g; conf.b = b; conf.sh = sh; conf.st = st;
  return 0;
}
int __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *sh, void **st) {
  *g = conf.g; *b = conf.b; *sh = conf.sh; *st = conf.st;
  return 0;
}
int hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t sh, void *st) {
  (void)b; (void)sh; (void)st;
  const char *name = "?";
  for (int k = 0; k < entries; ++k)
    if (table[k].key == f) name = table[k].name;
  if (stub_on_launch && stub_on_launch(name, g.x * g.y * g.z, args)) return last_error = 719;
  return 0;
}

int hipGetLastError(void) { const int e = last_error; last_error = 0; return e; }
const char *hipGetErrorString(int e) { return e ? "an error of the stand-in runtime" : "no error"; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int *v, int a, int d) { (void)a; (void)d; *v = 256; return 0; }
int hipGetSymbolAddress(void **p, const void *sym) {
  *p = NULL;
  for (int k = 0; k < entries; ++k)
    if (table[k].key == sym) *p = table[k].mem;
  return call("hipGetSymbolAddress");
}
int hipHostMalloc(void **p, size_t n, unsigned flags) {
  (void)flags;
  const int e = call("hipHostMalloc");
  *p = e ? NULL : calloc(1, n);
  return e;
}
int hipHostFree(void *p) { const int e = call("hipHostFree"); free(p); return e; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *st) {
  (void)kind; (void)st;
  const int e = call("hipMemcpyAsync");
  if (!e) memcpy(d, s, n);
  return e;
}
int hipMemsetAsync(void *d, int v, size_t n, void *st) {
  (void)st;
  const int e = call("hipMemsetAsync");
  if (!e) memset(d, v, n);
  return e;
}
int hipStreamSynchronize(void *st) { (void)st; return call("hipStreamSynchronize"); }
