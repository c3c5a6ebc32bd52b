/* A HIP runtime that runs nothing and writes down what it is asked: loaded ahead of libhmc.so
 * it answers the library's calls, so that the host side (which kernels go to which stream, how
 * streams fork and join, what happens when a call fails) can be tested without a GPU.
 * Device memory is host memory; a copy to the host yields ones, since no kernel fills it. */
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3;
typedef int err;

static char* text;
static size_t used, room;
static const char* fail_call = "";
static int fail_in;

#define LOG(...)                                                       \
  do {                                                                 \
    char line_[512];                                                   \
    int n_ = snprintf(line_, sizeof(line_), __VA_ARGS__);              \
    if (used + n_ + 2 > room) text = realloc(text, room = 2 * (used + n_ + 2)); \
    memcpy(text + used, line_, n_);                                    \
    used += n_;                                                        \
    text[used++] = '\n';                                               \
    text[used] = 0;                                                    \
  } while (0)

const char* record_text(void) { return text ? text : ""; }
void record_clear(void) {
  used = 0;
  if (text) text[0] = 0;
}
/* the nth call of `call` from now on fails, once */
void record_fail(const char* call, int nth) {
  fail_call = strdup(call);
  fail_in = nth;
}
static err status(const char* call) { return fail_in > 0 && !strcmp(call, fail_call) && --fail_in == 0 ? 1 : 0; }

/* ------------------------------------------------------------------ kernels */
static struct { const void* host; const char* name; } kernels[4096];
static int nkernels;
static struct { dim3 grid, block; size_t lds; void* stream; } config;

void** __hipRegisterFatBinary(const void* data) {
  static void* handle;
  (void)data;
  return &handle;
}
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterFunction(void** m, const void* host, char* dev, const char* name, unsigned lim, void* a, void* b,
                           dim3* c, dim3* d, int* e) {
  (void)m, (void)dev, (void)lim, (void)a, (void)b, (void)c, (void)d, (void)e;
  if (nkernels < 4096) {
    kernels[nkernels].host = host;
    kernels[nkernels++].name = strdup(name);
  }
}
void __hipRegisterVar(void** m, void* host, char* dev, char* name, int ext, size_t size, int c, int global) {
  (void)m, (void)host, (void)dev, (void)name, (void)ext, (void)size, (void)c, (void)global;
}
err __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void* stream) {
  config.grid = grid;
  config.block = block;
  config.lds = lds;
  config.stream = stream;
  return 0;
}
err __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, void** stream) {
  *grid = config.grid;
  *block = config.block;
  *lds = config.lds;
  *stream = config.stream;
  return 0;
}
err hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t lds, void* stream) {
  const char* name = "?";
  (void)block, (void)args, (void)lds;
  for (int i = 0; i < nkernels; ++i)
    if (kernels[i].host == f) name = kernels[i].name;
  LOG("launch %lld %u %s", (long long)(intptr_t)stream, grid.x, name);
  return 0;
}
err hipGetLastError(void) { return status("hipGetLastError"); }
const char* hipGetErrorString(err e) { return e ? "refused" : "ok"; }

/* ------------------------------------------------------------------ memory */
err hipMalloc(void** p, size_t n) {
  *p = calloc(1, n ? n : 1);
  return status("hipMalloc");
}
err hipFree(void* p) {
  free(p);
  return 0;
}
err hipHostMalloc(void** p, size_t n, unsigned flags) {
  (void)flags;
  return hipMalloc(p, n);
}
err hipHostFree(void* p) { return hipFree(p); }
static err copy(void* dst, const void* src, size_t n, int kind) {
  LOG("copy %d %zu", kind, n);
  if (kind == 1) memcpy(dst, src, n); /* host to device */
  if (kind == 2)
    for (size_t i = 0; i < n / 8; ++i) ((double*)dst)[i] = 1.0;
  return 0;
}
err hipMemcpy(void* dst, const void* src, size_t n, int kind) { return copy(dst, src, n, kind); }
err hipMemcpyAsync(void* dst, const void* src, size_t n, int kind, void* stream) {
  (void)stream;
  return copy(dst, src, n, kind);
}
err hipGetSymbolAddress(void** p, const void* s) {
  (void)s;
  *p = 0;
  return 1;
}

/* ------------------------------------------------------------------ device, streams, events, graphs */
static int compute_units = 256;
void record_compute_units(int n) { compute_units = n; }
err hipGetDevice(int* d) {
  *d = 0;
  return 0;
}
err hipDeviceGetAttribute(int* v, int attr, int dev) {
  (void)attr, (void)dev;
  *v = compute_units;
  return 0;
}
static intptr_t handles = 1000;
err hipStreamCreateWithFlags(void** s, unsigned flags) {
  (void)flags;
  *s = (void*)++handles;
  return status("hipStreamCreateWithFlags");
}
err hipStreamDestroy(void* s) {
  LOG("destroy %lld", (long long)(intptr_t)s);
  return 0;
}
err hipStreamSynchronize(void* s) {
  LOG("sync %lld", (long long)(intptr_t)s);
  return 0;
}
err hipEventCreateWithFlags(void** e, unsigned flags) {
  (void)flags;
  *e = (void*)++handles;
  return status("hipEventCreateWithFlags");
}
err hipEventCreate(void** e) { return hipEventCreateWithFlags(e, 0); }
err hipEventDestroy(void* e) {
  (void)e;
  return 0;
}
err hipEventRecord(void* e, void* s) {
  err st = status("hipEventRecord");
  if (!st) LOG("record %lld %lld", (long long)(intptr_t)s, (long long)(intptr_t)e);
  return st;
}
err hipStreamWaitEvent(void* s, void* e, unsigned flags) {
  err st = status("hipStreamWaitEvent");
  (void)flags;
  if (!st) LOG("wait %lld %lld", (long long)(intptr_t)s, (long long)(intptr_t)e);
  return st;
}
err hipEventSynchronize(void* e) {
  (void)e;
  return 0;
}
err hipEventElapsedTime(float* ms, void* a, void* b) {
  static int calls;
  (void)a, (void)b;
  *ms = 1.f / ++calls; /* each measurement faster than the one before */
  return 0;
}
err hipStreamBeginCapture(void* s, int mode) {
  (void)mode;
  LOG("capture %lld", (long long)(intptr_t)s);
  return 0;
}
err hipStreamEndCapture(void* s, void** g) {
  LOG("captured %lld", (long long)(intptr_t)s);
  *g = (void*)++handles;
  return 0;
}
err hipGraphInstantiate(void** x, void* g, void* n, char* log, size_t size) {
  (void)g, (void)n, (void)log, (void)size;
  *x = (void*)++handles;
  return 0;
}
err hipGraphLaunch(void* x, void* s) {
  LOG("replay %lld %lld", (long long)(intptr_t)s, (long long)(intptr_t)x);
  return 0;
}
err hipGraphDestroy(void* g) {
  (void)g;
  return 0;
}
err hipGraphExecDestroy(void* x) {
  (void)x;
  return 0;
}
