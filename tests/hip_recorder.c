/* A stand-in for the HIP runtime that runs nothing: it records kernel launches,
 * event records and stream waits, so that a test without a GPU can look at what a
 * call enqueues (loaded before the library, see recorder.py).  Memory is host
 * memory, copies are made, device copies and fills are not. */
#define _GNU_SOURCE
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>

typedef struct { uint32_t x, y, z; } dim3_;
enum { kMaxRec = 1 << 16, kMaxFn = 4096 };
static struct { const void* host; const char* name; } fns[kMaxFn];
static int n_fns;
static char* recs[kMaxRec];
static int n_recs;
static long launches, fail_at = -1;
static int last_error;
static uintptr_t next_handle = 0x1000;

static void rec(const char* fmt, ...);
#include <stdarg.h>
static void rec(const char* fmt, ...) {
  if (n_recs >= kMaxRec) return;
  va_list ap;
  va_start(ap, fmt);
  if (vasprintf(&recs[n_recs], fmt, ap) >= 0) ++n_recs;
  va_end(ap);
}
/* the test's side */
int rec_count(void) { return n_recs; }
const char* rec_get(int i) { return i < n_recs ? recs[i] : ""; }
void rec_clear(void) {
  for (int i = 0; i < n_recs; ++i) free(recs[i]);
  n_recs = 0;
  launches = 0;
}
void rec_fail_at(long launch) { fail_at = launch; launches = 0; }   /* this launch from now on fails */

/* registration */
void** __hipRegisterFatBinary(const void* data) { (void)data; return (void**)&next_handle; }
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterVar(void** m, void* v, char* h, char* d, int e, size_t s, int c, int g) {
  (void)m; (void)v; (void)h; (void)d; (void)e; (void)s; (void)c; (void)g;
}
void __hipRegisterFunction(void** m, const void* host, char* dev, const char* name, unsigned t, void* a, void* b,
                           void* c, void* d, int* w) {
  (void)m; (void)dev; (void)t; (void)a; (void)b; (void)c; (void)d; (void)w;
  if (n_fns < kMaxFn) { fns[n_fns].host = host; fns[n_fns++].name = strdup(name); }
}
static struct { dim3_ g, b; size_t lds; void* st; } cfg;
int __hipPushCallConfiguration(dim3_ g, dim3_ b, size_t lds, void* st) {
  cfg.g = g; cfg.b = b; cfg.lds = lds; cfg.st = st;
  return 0;
}
int __hipPopCallConfiguration(dim3_* g, dim3_* b, size_t* lds, void** st) {
  *g = cfg.g; *b = cfg.b; *lds = cfg.lds; *st = cfg.st;
  return 0;
}
int hipLaunchKernel(const void* f, dim3_ g, dim3_ b, void** args, size_t lds, void* st) {
  (void)args;
  if (fail_at >= 0 && launches++ == fail_at) {
    rec("fail");
    return last_error = 719;
  }
  const char* name = "?";
  for (int i = 0; i < n_fns; ++i)
    if (fns[i].host == f) name = fns[i].name;
  rec("launch %s %u,%u,%u %u,%u,%u %zu %p", name, g.x, g.y, g.z, b.x, b.y, b.z, lds, st);
  return 0;
}
int hipExtLaunchKernel(const void* f, dim3_ g, dim3_ b, void** args, size_t lds, void* st, void* e0, void* e1, int fl) {
  (void)e0; (void)e1; (void)fl;
  return hipLaunchKernel(f, g, b, args, lds, st);
}
int hipGetLastError(void) { int e = last_error; last_error = 0; return e; }
const char* hipGetErrorString(int e) { return e ? "error" : "no error"; }

/* memory: pages are committed when touched */
int hipMalloc(void** p, size_t n) {
  *p = mmap(NULL, n + 4096, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  return *p == MAP_FAILED ? 2 : 0;
}
int hipFree(void* p) { (void)p; return 0; }
int hipMemcpy(void* d, const void* s, size_t n, int k) { (void)k; memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int k, void* st) {
  if (k == 1) memcpy(d, s, n);
  rec("copy %zu %p", n, st);
  return 0;
}
int hipMemcpy2DAsync(void* d, size_t dp, const void* s, size_t sp, size_t w, size_t h, int k, void* st) {
  (void)d; (void)dp; (void)s; (void)sp; (void)k;
  rec("copy %zu %p", w * h, st);
  return 0;
}
int hipMemset(void* d, int v, size_t n) { (void)d; (void)v; (void)n; return 0; }
int hipMemsetAsync(void* d, int v, size_t n, void* st) { (void)d; (void)v; (void)n; (void)st; return 0; }
int hipGetSymbolAddress(void** p, const void* s) { (void)s; return hipMalloc(p, (size_t)32 << 20); }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipDeviceSynchronize(void) { return 0; }

/* streams, events, graphs: numbers */
static int handle(void** h) { *h = (void*)(next_handle += 0x10); return 0; }
int hipStreamCreateWithFlags(void** s, unsigned f) { (void)f; return handle(s); }
int hipStreamDestroy(void* s) { (void)s; return 0; }
int hipStreamSynchronize(void* s) { (void)s; return 0; }
int hipStreamWaitEvent(void* s, void* e, unsigned f) { (void)f; rec("wait %p %p", s, e); return 0; }
int hipEventCreate(void** e) { return handle(e); }
int hipEventCreateWithFlags(void** e, unsigned f) { (void)f; return handle(e); }
int hipEventDestroy(void* e) { (void)e; return 0; }
int hipEventRecord(void* e, void* s) { rec("record %p %p", e, s); return 0; }
int hipEventSynchronize(void* e) { (void)e; return 0; }
int hipEventElapsedTime(float* ms, void* a, void* b) { (void)a; (void)b; *ms = 0.0f; return 0; }
int hipStreamBeginCapture(void* s, int m) { (void)m; rec("capture %p", s); return 0; }
int hipStreamEndCapture(void* s, void** g) { rec("captured %p", s); return handle(g); }
int hipGraphInstantiate(void** x, void* g, void* a, void* b, size_t c) { (void)g; (void)a; (void)b; (void)c; return handle(x); }
int hipGraphLaunch(void* g, void* s) { rec("graph %p %p", g, s); return 0; }
int hipGraphDestroy(void* g) { (void)g; return 0; }
int hipGraphExecDestroy(void* g) { (void)g; return 0; }
