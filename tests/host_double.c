/* A host double of the HIP runtime calls that liblbm.so makes, for tests of its host code on a
 * machine without a GPU.  Loaded with RTLD_GLOBAL before the library, whose calls then bind to it.
 * "Device" memory is host memory, kernels are not run: every launch is reported to a callback, which
 * may make it fail.  Copies between device buffers are reported and not made. */
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;
typedef int (*launch_cb)(const char* kernel, uint32_t gx, uint32_t gy, uint32_t gz, uint32_t threads, void** args);
typedef void (*call_cb)(const char* call, void* dst, const void* src, size_t bytes);

enum { MAX_KERNELS = 1024, NOT_PERMITTED_IN_CAPTURE = 900 };
static struct { const void* host; const char* name; } kernels[MAX_KERNELS];
static int n_kernels, last_error, capturing;
static launch_cb on_launch;
static call_cb on_call;
static dim3_t cfg_grid, cfg_block;
static size_t cfg_lds;
static void* cfg_stream;
static char symbol_memory[8 << 20];

void double_callbacks(launch_cb l, call_cb c) { on_launch = l; on_call = c; }
void double_capturing(int on) { capturing = on; }

static void say(const char* call, void* dst, const void* src, size_t bytes) {
  if (on_call) on_call(call, dst, src, bytes);
}
static int result(int e) {
  if (e) last_error = e;
  return e;
}

void** __hipRegisterFatBinary(const void* d) { (void)d; return (void**)symbol_memory; }
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterFunction(void** m, const void* host, char* dev, const char* name, unsigned n, void* a, void* b,
                           void* c, void* d, int* w) {
  (void)m; (void)dev; (void)n; (void)a; (void)b; (void)c; (void)d; (void)w;
  if (n_kernels < MAX_KERNELS) {
    kernels[n_kernels].host = host;
    kernels[n_kernels++].name = name;
  }
}
void __hipRegisterVar(void** m, void* v, char* h, char* d, int e, size_t s, int c, int g) {
  (void)m; (void)v; (void)h; (void)d; (void)e; (void)s; (void)c; (void)g;
}
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t lds, void* s) {
  cfg_grid = g; cfg_block = b; cfg_lds = lds; cfg_stream = s;
  return 0;
}
int __hipPopCallConfiguration(dim3_t* g, dim3_t* b, size_t* lds, void** s) {
  *g = cfg_grid; *b = cfg_block; *lds = cfg_lds; *s = cfg_stream;
  return 0;
}
int hipLaunchKernel(const void* f, dim3_t g, dim3_t b, void** args, size_t lds, void* s) {
  const char* name = "?";
  (void)lds; (void)s;
  for (int i = 0; i < n_kernels; ++i)
    if (kernels[i].host == f) name = kernels[i].name;
  return result(on_launch ? on_launch(name, g.x, g.y, g.z, b.x * b.y * b.z, args) : 0);
}
int hipGetLastError(void) {  /* returns the error and clears it, as the runtime does */
  const int e = last_error;
  last_error = 0;
  return e;
}
int hipPeekAtLastError(void) { return last_error; }

int hipMalloc(void** p, size_t n) {
  say("hipMalloc", 0, 0, n);
  return (*p = calloc(1, n ? n : 1)) ? 0 : result(2);
}
int hipFree(void* p) { free(p); return 0; }
int hipGetSymbolAddress(void** p, const void* s) { (void)s; *p = symbol_memory; return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
static int copy(const char* call, void* d, const void* s, size_t n, int kind) {
  say(call, d, s, n);
  if (kind == 1 || kind == 2) memcpy(d, s, n);
  return 0;
}
int hipMemcpy(void* d, const void* s, size_t n, int kind) { return copy("hipMemcpy", d, s, n, kind); }
int hipMemcpyAsync(void* d, const void* s, size_t n, int kind, void* st) {
  (void)st;
  return copy("hipMemcpyAsync", d, s, n, kind);
}
int hipMemset(void* d, int v, size_t n) { say("hipMemset", d, 0, n); memset(d, v, n); return 0; }
int hipMemsetAsync(void* d, int v, size_t n, void* st) {
  (void)st;
  say("hipMemsetAsync", d, 0, n);
  memset(d, v, n);
  return 0;
}
int hipStreamSynchronize(void* s) {
  (void)s;
  say("hipStreamSynchronize", 0, 0, 0);
  return result(capturing ? NOT_PERMITTED_IN_CAPTURE : 0);
}
int hipStreamIsCapturing(void* s, int* status) { (void)s; *status = capturing; return 0; }
int hipEventCreate(void** e) { *e = malloc(1); return 0; }
int hipEventDestroy(void* e) { free(e); return 0; }
int hipEventRecord(void* e, void* s) { (void)e; (void)s; return 0; }
int hipEventSynchronize(void* e) { (void)e; return 0; }
int hipEventElapsedTime(float* ms, void* a, void* b) { (void)a; (void)b; *ms = 0.f; return 0; }
