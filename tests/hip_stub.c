/* The HIP runtime calls that liblbm makes, on the CPU: "device" memory is host memory, copies are done at once, kernels
 * are counted and not run, and a chosen launch can be made to fail.  For tests of the library's host side. */
#include <pthread.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <time.h>

typedef int err;
enum { OK = 0, LAUNCH_FAILURE = 719 };
typedef struct {
  unsigned x, y, z;
} dim;

static pthread_mutex_t mu = PTHREAD_MUTEX_INITIALIZER;
static __thread err last_error;
static struct {
  const void* fn;
  const char* name;
  long count;
} kernels[512];
static int nkernels;
static long launches, fail_first = -1, fail_count, host_allocs, host_live;
static dim last_grid;
static unsigned fast_grid;
static int last_int;

/* ---- for the tests */
void stub_reset(void) {
  pthread_mutex_lock(&mu);
  for (int i = 0; i < nkernels; ++i) kernels[i].count = 0;
  launches = 0;
  fail_first = -1;
  pthread_mutex_unlock(&mu);
}
/* launches number first .. first + count - 1 after the last reset fail */
void stub_fail(long first, long count) { fail_first = first, fail_count = count; }
/* launches of the kernels whose mangled name contains `part` */
long stub_launched(const char* part) {
  long n = 0;
  for (int i = 0; i < nkernels; ++i)
    if (strstr(kernels[i].name, part)) n += kernels[i].count;
  return n;
}
unsigned stub_last_grid(void) { return last_grid.x; }
/* events say that time passes ten times as fast after a launch of so many workgroups */
void stub_fast_grid(unsigned n) { fast_grid = n; }
/* first argument of the last launch, where that is an int */
int stub_last_int(void) { return last_int; }
long stub_host_allocs(void) { return host_allocs; }
long stub_host_live(void) { return host_live; }

/* ---- modules and launches */
void** __hipRegisterFatBinary(const void* data) {
  static void* handle;
  (void)data;
  return &handle;
}
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterFunction(void** m, const void* fn, char* dev, const char* name, unsigned limit, void* a, void* b, void* c,
                           void* d, int* e) {
  (void)m, (void)dev, (void)limit, (void)a, (void)b, (void)c, (void)d, (void)e;
  if (nkernels < 512) {
    kernels[nkernels].fn = fn;
    kernels[nkernels++].name = strdup(name);
  }
}
void __hipRegisterVar(void** m, void* var, char* h, char* d, int ext, size_t size, int constant, int global) {
  (void)m, (void)var, (void)h, (void)d, (void)ext, (void)size, (void)constant, (void)global;
}
static __thread struct {
  dim grid, block;
  size_t shared;
  void* stream;
} config;
err __hipPushCallConfiguration(dim grid, dim block, size_t shared, void* stream) {
  config.grid = grid, config.block = block, config.shared = shared, config.stream = stream;
  return OK;
}
err __hipPopCallConfiguration(dim* grid, dim* block, size_t* shared, void** stream) {
  *grid = config.grid, *block = config.block, *shared = config.shared, *stream = config.stream;
  return OK;
}
err hipLaunchKernel(const void* fn, dim grid, dim block, void** args, size_t shared, void* stream) {
  (void)block, (void)shared, (void)stream;
  pthread_mutex_lock(&mu);
  const long at = launches++;
  const int bad = fail_first >= 0 && at >= fail_first && at < fail_first + fail_count;
  last_grid = grid;
  last_int = *(const int*)args[0];
  for (int i = 0; i < nkernels && !bad; ++i)
    if (kernels[i].fn == fn) ++kernels[i].count;
  pthread_mutex_unlock(&mu);
  if (bad) last_error = LAUNCH_FAILURE;
  return bad ? LAUNCH_FAILURE : OK;
}
err hipGetLastError(void) {
  const err e = last_error;
  last_error = OK;
  return e;
}
const char* hipGetErrorString(err e) { return e == OK ? "no error" : "launch failure"; }

/* ---- memory */
err hipHostMalloc(void** p, size_t bytes, unsigned flags) {
  (void)flags;
  pthread_mutex_lock(&mu);
  ++host_allocs;
  ++host_live;
  pthread_mutex_unlock(&mu);
  *p = calloc(1, bytes);
  return OK;
}
err hipHostFree(void* p) {
  pthread_mutex_lock(&mu);
  --host_live;
  pthread_mutex_unlock(&mu);
  free(p);
  return OK;
}
err hipMemcpyAsync(void* to, const void* from, size_t bytes, int kind, void* stream) {
  (void)kind, (void)stream;
  memcpy(to, from, bytes);
  return OK;
}
err hipMemsetAsync(void* to, int value, size_t bytes, void* stream) {
  (void)stream;
  memset(to, value, bytes);
  return OK;
}
err hipGetSymbolAddress(void** p, const void* symbol) {
  static char scratch[16 << 20] __attribute__((aligned(256)));
  (void)symbol;
  *p = scratch;
  return OK;
}
err hipGetDevice(int* d) {
  *d = 0;
  return OK;
}

/* ---- streams, events, graphs: waiting takes a moment, so that calls of several threads overlap */
static void moment(void) {
  const struct timespec t = {0, 50000};
  nanosleep(&t, NULL);
}
err hipStreamSynchronize(void* s) {
  (void)s;
  moment();
  return OK;
}
err hipStreamBeginCapture(void* s, int mode) {
  (void)s, (void)mode;
  return OK;
}
err hipStreamEndCapture(void* s, void** g) {
  (void)s;
  *g = malloc(1);
  return OK;
}
err hipGraphInstantiate(void** x, void* g, void** node, char* log, size_t n) {
  (void)g, (void)node, (void)log, (void)n;
  *x = malloc(1);
  return OK;
}
err hipGraphLaunch(void* x, void* s) {
  (void)x, (void)s;
  return OK;
}
err hipGraphDestroy(void* g) {
  free(g);
  return OK;
}
err hipGraphExecDestroy(void* x) {
  free(x);
  return OK;
}
err hipEventCreate(void** e) {
  *e = malloc(1);
  return OK;
}
err hipEventCreateWithFlags(void** e, unsigned flags) {
  (void)flags;
  *e = malloc(1);
  return OK;
}
err hipEventDestroy(void* e) {
  free(e);
  return OK;
}
err hipEventRecord(void* e, void* s) {
  (void)e, (void)s;
  return OK;
}
err hipEventSynchronize(void* e) {
  (void)e;
  moment();
  return OK;
}
err hipEventElapsedTime(float* ms, void* a, void* b) {
  (void)a, (void)b;
  *ms = fast_grid && last_grid.x == fast_grid ? 0.1f : 1.0f;
  return OK;
}
int roctxRangePushA(const char* s) {
  (void)s;
  return 0;
}
int roctxRangePop(void) { return 0; }
