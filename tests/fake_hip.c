/* A HIP runtime without a device, for CPU tests of the library's host code: memory is
 * reserved address space that reads as zeros (with a limit on what is held at once),
 * kernels do nothing and are recorded, streams are always idle.  Loaded before libdd.so
 * with its symbols global, so that the library binds to it. */
#define _GNU_SOURCE
#include <pthread.h>
#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>

typedef int err_t;
enum { OK = 0, INVALID = 1, OOM = 2 };
typedef struct { unsigned x, y, z; } d3;

static pthread_mutex_t mu = PTHREAD_MUTEX_INITIALIZER;

/* ---- device memory ---- */
#define MAX_BLOCKS 65536
static struct { char* p; size_t n; } blocks[MAX_BLOCKS];
static size_t live, peak, limit = (size_t)1 << 40;
static long n_blocks, refused, frees;

static err_t take(void** p, size_t n) {
  err_t e = OOM;
  pthread_mutex_lock(&mu);
  size_t map = n ? n : 1;
  if (live + map <= limit && n_blocks < MAX_BLOCKS) {
    void* a = mmap(NULL, map, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (a != MAP_FAILED) {
      blocks[n_blocks].p = a;
      blocks[n_blocks++].n = map;
      live += map;
      if (live > peak) peak = live;
      *p = a;
      e = OK;
    }
  }
  if (e) ++refused;
  pthread_mutex_unlock(&mu);
  return e;
}
static err_t give(void* p) {
  err_t e = p ? INVALID : OK;
  pthread_mutex_lock(&mu);
  for (long i = 0; p && i < n_blocks; ++i)
    if (blocks[i].p == p) {
      munmap(p, blocks[i].n);
      live -= blocks[i].n;
      blocks[i] = blocks[--n_blocks];
      ++frees;
      e = OK;
      break;
    }
  pthread_mutex_unlock(&mu);
  return e;
}
size_t fake_live(void) { return live; }
size_t fake_peak(void) { size_t v = peak; peak = live; return v; }
long fake_refused(void) { return refused; }
void fake_limit(size_t n) { limit = n; }

err_t hipMalloc(void** p, size_t n) { return take(p, n); }
err_t hipFree(void* p) { return give(p); }
err_t hipMallocAsync(void** p, size_t n, void* st) { (void)st; return take(p, n); }
err_t hipFreeAsync(void* p, void* st) { (void)st; return give(p); }
err_t hipHostMalloc(void** p, size_t n, unsigned f) { (void)f; *p = calloc(1, n); return *p ? OK : OOM; }
err_t hipHostFree(void* p) { free(p); return OK; }
err_t hipMemGetInfo(size_t* f, size_t* t) { *f = limit - live; *t = limit; return OK; }

/* ---- kernels ---- */
static struct { const void* f; const char* name; } kernels[1024];
static int n_kernels;
static struct { const char* name; d3 grid; uint64_t arg[8]; } launches[1 << 16];
static long n_launches;
static char watch[64];
static int watch_size[8], n_watch;
static __thread const char* last_kernel = "";
static int word_value = -1;
static char word_kernel[64];

void** __hipRegisterFatBinary(const void* d) { (void)d; static void* h; return &h; }
void __hipUnregisterFatBinary(void** h) { (void)h; }
void __hipRegisterFunction(void** h, const void* f, char* df, const char* name, unsigned tl, void* a, void* b,
                           void* c, void* d, int* w) {
  (void)h, (void)df, (void)tl, (void)a, (void)b, (void)c, (void)d, (void)w;
  if (n_kernels < 1024) kernels[n_kernels].f = f, kernels[n_kernels++].name = name;
}
void __hipRegisterVar(void** h, void* v, char* hv, char* dv, int e, size_t s, int c, int g) {
  (void)h, (void)v, (void)hv, (void)dv, (void)e, (void)s, (void)c, (void)g;
}
static __thread struct { d3 g, b; size_t s; void* st; } conf;
err_t __hipPushCallConfiguration(d3 g, d3 b, size_t s, void* st) {
  conf.g = g, conf.b = b, conf.s = s, conf.st = st;
  return OK;
}
err_t __hipPopCallConfiguration(d3* g, d3* b, size_t* s, void** st) {
  *g = conf.g, *b = conf.b, *s = conf.s, *st = conf.st;
  return OK;
}
err_t hipLaunchKernel(const void* f, d3 g, d3 b, void** args, size_t s, void* st) {
  (void)b, (void)s, (void)st;
  const char* name = "?";
  for (int i = 0; i < n_kernels; ++i)
    if (kernels[i].f == f) name = kernels[i].name;
  last_kernel = name;
  pthread_mutex_lock(&mu);
  if (n_launches < (1 << 16)) {
    launches[n_launches].name = name;
    launches[n_launches].grid = g;
    if (n_watch && strstr(name, watch))
      for (int i = 0; i < n_watch; ++i) memcpy(&launches[n_launches].arg[i], args[i], watch_size[i]);
    ++n_launches;
  }
  pthread_mutex_unlock(&mu);
  return OK;
}
/* Forget the launches; from now on copy the first n arguments (their sizes) of kernels named so. */
void fake_watch(const char* name, int n, const int* sizes) {
  n_launches = 0;
  memset(launches, 0, sizeof launches);
  strncpy(watch, name, sizeof watch - 1);
  n_watch = n;
  for (int i = 0; i < n; ++i) watch_size[i] = sizes[i];
}
long fake_launches(const char* name) {
  long c = 0;
  for (long i = 0; i < n_launches; ++i) c += strstr(launches[i].name, name) != NULL;
  return c;
}
uint64_t fake_arg(const char* name, long k, int i) {
  for (long j = 0; j < n_launches; ++j)
    if (strstr(launches[j].name, name) && k-- == 0) return launches[j].arg[i];
  return 0;
}
/* A 4-byte read-back right after a kernel named so gives `value` (below 0: what is there). */
void fake_word(const char* kernel, int value) {
  strncpy(word_kernel, kernel, sizeof word_kernel - 1);
  word_value = value;
}

/* ---- copies, streams, events ---- */
static err_t copy(void* d, const void* s, size_t n, int kind) {
  if (kind == 2 && n == 4 && word_value >= 0 && strstr(last_kernel, word_kernel)) memcpy(d, &word_value, 4);
  else if (n) memcpy(d, s, n);
  return OK;
}
err_t hipMemcpy(void* d, const void* s, size_t n, int k) { return copy(d, s, n, k); }
err_t hipMemcpyAsync(void* d, const void* s, size_t n, int k, void* st) { (void)st; return copy(d, s, n, k); }
err_t hipMemcpy2DAsync(void* d, size_t dp, const void* s, size_t sp, size_t w, size_t h, int k, void* st) {
  (void)k, (void)st;
  for (size_t i = 0; i < h; ++i) memcpy((char*)d + i * dp, (const char*)s + i * sp, w);
  return OK;
}
err_t hipMemsetAsync(void* d, int v, size_t n, void* st) {
  (void)st;
  if (v) memset(d, v, n);   /* zeros are there already: nothing writes but copies of small results */
  return OK;
}
err_t hipGetSymbolAddress(void** p, const void* s) { (void)s; *p = NULL; return INVALID; }
err_t hipGetDevice(int* d) { *d = 0; return OK; }
err_t hipSetDevice(int d) { (void)d; return OK; }
err_t hipGetLastError(void) { return OK; }
const char* hipGetErrorString(err_t e) { return e == OOM ? "out of memory" : "error"; }
err_t hipDeviceSynchronize(void) { return OK; }
static char handle;
err_t hipStreamCreateWithFlags(void** s, unsigned f) { (void)f; *s = &handle; return OK; }
err_t hipStreamDestroy(void* s) { (void)s; return OK; }
err_t hipStreamSynchronize(void* s) { (void)s; return OK; }
err_t hipStreamWaitEvent(void* s, void* e, unsigned f) { (void)s, (void)e, (void)f; return OK; }
err_t hipThreadExchangeStreamCaptureMode(int* m) { (void)m; return OK; }
err_t hipEventCreate(void** e) { *e = &handle; return OK; }
err_t hipEventCreateWithFlags(void** e, unsigned f) { (void)f; *e = &handle; return OK; }
err_t hipEventDestroy(void* e) { (void)e; return OK; }
err_t hipEventRecord(void* e, void* s) { (void)e, (void)s; return OK; }
err_t hipEventQuery(void* e) { (void)e; return OK; }
err_t hipEventSynchronize(void* e) { (void)e; return OK; }
err_t hipEventElapsedTime(float* ms, void* a, void* b) { (void)a, (void)b; *ms = 0; return OK; }
err_t hipStreamBeginCapture(void* s, int m) { (void)s, (void)m; return INVALID; }
err_t hipStreamEndCapture(void* s, void** g) { (void)s; *g = NULL; return INVALID; }
err_t hipGraphInstantiate(void** e, void* g, void* a, char* b, size_t c) { (void)e, (void)g, (void)a, (void)b, (void)c; return INVALID; }
err_t hipGraphDestroy(void* g) { (void)g; return OK; }
err_t hipGraphExecDestroy(void* g) { (void)g; return OK; }
err_t hipGraphLaunch(void* g, void* s) { (void)g, (void)s; return INVALID; }
