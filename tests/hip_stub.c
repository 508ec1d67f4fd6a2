/* A stand-in for the HIP runtime calls that libweno_l2is.so makes, for tests
 * of its host side without a GPU: device memory is a range of addresses that
 * nothing dereferences (with a settable capacity), a kernel launch is checked
 * against the runtime's limits and written to a log, copies to the host give
 * zeros.  Loaded with RTLD_GLOBAL before the library. */
#include <stdarg.h>
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { unsigned x, y, z; } dim3_t;

enum { OK = 0, INVALID_VALUE = 1, OUT_OF_MEMORY = 2, INVALID_CONFIGURATION = 9 };

static char log_buf[1 << 20];
static size_t log_n;
static void note(const char *f, ...) {
  va_list a;
  va_start(a, f);
  const int k = vsnprintf(log_buf + log_n, sizeof log_buf - log_n, f, a);
  va_end(a);
  if (k > 0 && log_n + (size_t)k < sizeof log_buf) log_n += (size_t)k;
}
const char *stub_log(void) { return log_buf; }
void stub_clear(void) { log_n = 0; log_buf[0] = 0; }

/* device memory */
static size_t capacity = (size_t)1 << 62, used, peak;
static struct { uintptr_t p; size_t n; } mem[4096];
static int n_mem;
static uintptr_t next_addr = (uintptr_t)1 << 44;
void stub_capacity(size_t b) { capacity = b; peak = used; }
size_t stub_used(void) { return used; }
size_t stub_peak(void) { return peak; }

int hipMalloc(void **p, size_t n) {
  if (n > capacity || used > capacity - n || n_mem == 4096) return OUT_OF_MEMORY;
  mem[n_mem].p = next_addr;
  mem[n_mem++].n = n;
  *p = (void *)next_addr;
  next_addr += (n + 0xffffu) & ~(size_t)0xffff;
  used += n;
  if (used > peak) peak = used;
  return OK;
}
int hipFree(void *p) {
  for (int i = 0; i < n_mem; ++i)
    if (mem[i].p == (uintptr_t)p) {
      used -= mem[i].n;
      mem[i] = mem[--n_mem];
      break;
    }
  return OK;
}
int hipMemGetInfo(size_t *avail, size_t *total) {
  *avail = capacity - used;
  *total = capacity;
  return OK;
}
int hipHostMalloc(void **p, size_t n, unsigned flags) {
  (void)flags;
  return (*p = calloc(1, n ? n : 1)) ? OK : OUT_OF_MEMORY;
}
int hipHostFree(void *p) { free(p); return OK; }

/* kernels */
static struct { const void *f; const char *name; } fun[2048];
static int n_fun;
static struct { dim3_t g, b; size_t lds; void *s; } cfg;
static int last;

void **__hipRegisterFatBinary(const void *d) { (void)d; return (void **)&n_fun; }
void __hipUnregisterFatBinary(void **h) { (void)h; }
void __hipRegisterVar(void **h, ...) { (void)h; }
void __hipRegisterFunction(void **h, const void *f, char *dev, const char *name, ...) {
  (void)h;
  (void)dev;
  if (n_fun < 2048) {
    fun[n_fun].f = f;
    fun[n_fun++].name = name;
  }
}
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t lds, void *s) {
  cfg.g = g;
  cfg.b = b;
  cfg.lds = lds;
  cfg.s = s;
  return OK;
}
int __hipPopCallConfiguration(dim3_t *g, dim3_t *b, size_t *lds, void **s) {
  *g = cfg.g;
  *b = cfg.b;
  *lds = cfg.lds;
  *s = cfg.s;
  return OK;
}
int hipLaunchKernel(const void *f, dim3_t g, dim3_t b, void **args, size_t lds, void *s) {
  const char *name = "?";
  (void)args;
  (void)lds;
  (void)s;
  for (int i = 0; i < n_fun; ++i)
    if (fun[i].f == f) name = fun[i].name;
  note("launch %s %u %u %u %u\n", name, g.x, g.y, g.z, b.x * b.y * b.z);
  /* at most 2^32 - 1 work items along a dimension */
  if ((uint64_t)g.x * b.x > 0xffffffffull || (uint64_t)g.y * b.y > 0xffffffffull ||
      (uint64_t)g.z * b.z > 0xffffffffull || !g.x || !g.y || !g.z || g.y > 65536 || g.z > 65536)
    return last = INVALID_CONFIGURATION;
  return OK;
}
int hipGetLastError(void) {
  const int e = last;
  last = OK;
  return e;
}

/* copies, streams, events, graphs */
int hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *st) {
  (void)s;
  (void)st;
  if (kind == 2) memset(d, 0, n); /* device to host */
  return OK;
}
int hipMemcpy(void *d, const void *s, size_t n, int kind) { return hipMemcpyAsync(d, s, n, kind, 0); }
int hipMemsetAsync(void *d, int v, size_t n, void *st) {
  (void)d; (void)v; (void)n; (void)st;
  return OK;
}
int hipGetDevice(int *d) { *d = 0; return OK; }
int hipSetDevice(int d) { (void)d; return OK; }
int hipDeviceGetAttribute(int *v, int a, int d) { (void)a; (void)d; *v = 256; return OK; }
int hipGetSymbolAddress(void **p, const void *s) { (void)s; *p = (void *)((uintptr_t)1 << 43); return OK; }
int hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; *s = (void *)(uintptr_t)0x1000; return OK; }
int hipStreamDestroy(void *s) { (void)s; return OK; }
int hipStreamSynchronize(void *s) { (void)s; note("sync\n"); return OK; }
int hipStreamBeginCapture(void *s, int m) { (void)s; (void)m; note("capture\n"); return OK; }
int hipStreamEndCapture(void *s, void **g) { (void)s; *g = (void *)(uintptr_t)0x2000; return OK; }
static int capturing;
void stub_capturing(int on) { capturing = on; }
int hipStreamIsCapturing(void *s, int *status) { (void)s; *status = capturing; return OK; }
static uintptr_t n_exec;
int hipGraphInstantiate(void **e, void *g, void **n, char *l, size_t z) {
  (void)g; (void)n; (void)l; (void)z;
  *e = (void *)(0x3000 + ++n_exec);
  note("instantiate %d\n", (int)n_exec);
  return OK;
}
int hipGraphLaunch(void *e, void *s) { (void)s; note("graph %d\n", (int)((uintptr_t)e - 0x3000)); return OK; }
int hipGraphExecDestroy(void *e) { note("destroy %d\n", (int)((uintptr_t)e - 0x3000)); return OK; }
int hipGraphDestroy(void *g) { (void)g; return OK; }
int hipEventCreate(void **e) { *e = (void *)(uintptr_t)0x4000; return OK; }
int hipEventCreateWithFlags(void **e, unsigned f) { (void)f; return hipEventCreate(e); }
int hipEventDestroy(void *e) { (void)e; return OK; }
int hipEventRecord(void *e, void *s) { (void)e; (void)s; return OK; }
int hipEventQuery(void *e) { (void)e; return OK; }
int hipEventSynchronize(void *e) { (void)e; note("event_sync\n"); return OK; }
int hipEventElapsedTime(float *t, void *a, void *b) { (void)a; (void)b; *t = 0.f; return OK; }
