/* A HIP runtime that runs nothing, for tests of the library's host code
 * without a GPU (test_host_runtime.py loads it before libdsi.so, so that the
 * library's calls come here).  Device memory is address space without access;
 * a budget makes allocations fail; a launch writes one line to a log: kernel
 * name, grid and block.  While `capturing` is set, allocating and freeing fail,
 * as they do on a stream that is being captured. */
#define _GNU_SOURCE
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>

typedef struct { uint32_t x, y, z; } dim3_t;

enum { SUCCESS = 0, OUT_OF_MEMORY = 2, INVALID_VALUE = 1, CAPTURE_UNSUPPORTED = 900 };

static struct { void* p; size_t n; } blocks[1 << 16];
static int n_blocks;
static size_t in_use, budget = (size_t)1 << 46;
static int capturing, mallocs, frees, refused;
static char* text;
static size_t text_len, text_cap;
static struct { const void* f; const char* name; } kernels[8192];
static int n_kernels;
static dim3_t cfg_grid, cfg_block;

void stub_budget(size_t free_bytes) { budget = in_use + free_bytes; }
void stub_capture(int on) { capturing = on; }
size_t stub_in_use(void) { return in_use; }
int stub_mallocs(void) { return mallocs; }
int stub_frees(void) { return frees; }
int stub_refused(void) { return refused; }
const char* stub_log(void) { return text ? text : ""; }
int stub_kernels(void) { return n_kernels; }
const char* stub_kernel(int i) { return kernels[i].name; }
void stub_clear(void) {
  mallocs = frees = refused = 0;
  text_len = 0;
  if (text) text[0] = 0;
}

int hipMalloc(void** p, size_t n) {
  *p = NULL;
  if (capturing) return ++refused, CAPTURE_UNSUPPORTED;
  n = (n + 4095) & ~(size_t)4095;
  if (in_use + n > budget || n_blocks == 1 << 16) return ++refused, OUT_OF_MEMORY;
  void* q = mmap(NULL, n, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  if (q == MAP_FAILED) return OUT_OF_MEMORY;
  blocks[n_blocks].p = q;
  blocks[n_blocks++].n = n;
  in_use += n;
  ++mallocs;
  *p = q;
  return SUCCESS;
}
int hipFree(void* p) {
  if (!p) return SUCCESS;
  if (capturing) return CAPTURE_UNSUPPORTED;
  for (int i = 0; i < n_blocks; ++i)
    if (blocks[i].p == p) {
      munmap(p, blocks[i].n);
      in_use -= blocks[i].n;
      blocks[i] = blocks[--n_blocks];
      ++frees;
      return SUCCESS;
    }
  fprintf(stderr, "hipFree of %p, which is not allocated\n", p);
  abort();
}
int hipMemGetInfo(size_t* avail, size_t* total) { *avail = budget - in_use; *total = budget; return SUCCESS; }
int hipMemset(void* p, int v, size_t n) { (void)p; (void)v; (void)n; return SUCCESS; }
int hipMemcpy(void* d, const void* s, size_t n, int kind) {
  (void)s;
  if (kind == 2) memset(d, 0, n);   /* device to host */
  return SUCCESS;
}
int hipMemcpyAsync(void* d, const void* s, size_t n, int kind, void* st) { (void)st; return hipMemcpy(d, s, n, kind); }
int hipDeviceSynchronize(void) { return SUCCESS; }
int hipStreamSynchronize(void* s) { (void)s; return SUCCESS; }
int hipGetDevice(int* d) { *d = 0; return SUCCESS; }
int hipGetLastError(void) { return SUCCESS; }
const char* hipGetErrorString(int e) { return e ? "stub error" : "no error"; }
int hipGetSymbolAddress(void** p, const void* s) { *p = (void*)s; return SUCCESS; }
int hipEventCreate(void** e) { *e = (void*)1; return SUCCESS; }
int hipEventDestroy(void* e) { (void)e; return SUCCESS; }
int hipEventRecord(void* e, void* s) { (void)e; (void)s; return SUCCESS; }
int hipEventSynchronize(void* e) { (void)e; return SUCCESS; }
int hipEventElapsedTime(float* ms, void* a, void* b) { (void)a; (void)b; *ms = 1.f; return SUCCESS; }
int hipStreamIsCapturing(void* s, int* st) { (void)s; *st = capturing ? 1 : 0; return SUCCESS; }
int hipStreamBeginCapture(void* s, int mode) { (void)s; (void)mode; if (capturing) return INVALID_VALUE; capturing = 1; return SUCCESS; }
int hipStreamEndCapture(void* s, void** g) { (void)s; capturing = 0; *g = (void*)1; return SUCCESS; }
int hipGraphInstantiate(void** x, void* g, void* n, char* l, size_t b) { (void)g; (void)n; (void)l; (void)b; *x = (void*)1; return SUCCESS; }
int hipGraphDestroy(void* g) { (void)g; return SUCCESS; }
int hipGraphExecDestroy(void* x) { (void)x; return SUCCESS; }
int hipGraphLaunch(void* x, void* s) { (void)x; (void)s; return SUCCESS; }

void** __hipRegisterFatBinary(const void* d) { (void)d; static void* h; return &h; }
void __hipUnregisterFatBinary(void** h) { (void)h; }
void __hipRegisterVar(void** m, void* v, char* h, char* d, int e, size_t n, int c, int g) {
  (void)m; (void)v; (void)h; (void)d; (void)e; (void)n; (void)c; (void)g;
}
void __hipRegisterFunction(void** m, const void* host, char* dev, const char* name, unsigned t, void* a, void* b, void* c,
                           void* d, int* w) {
  (void)m; (void)dev; (void)t; (void)a; (void)b; (void)c; (void)d; (void)w;
  if (n_kernels < (int)(sizeof kernels / sizeof kernels[0])) {
    kernels[n_kernels].f = host;
    kernels[n_kernels++].name = name;
  }
}
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t lds, void* s) {
  (void)lds; (void)s;
  cfg_grid = g;
  cfg_block = b;
  return SUCCESS;
}
int __hipPopCallConfiguration(dim3_t* g, dim3_t* b, size_t* lds, void** s) {
  *g = cfg_grid;
  *b = cfg_block;
  *lds = 0;
  *s = NULL;
  return SUCCESS;
}
int hipLaunchKernel(const void* f, dim3_t g, dim3_t b, void** args, size_t lds, void* s) {
  (void)args; (void)lds; (void)s;
  const char* name = "?";
  for (int i = 0; i < n_kernels; ++i)
    if (kernels[i].f == f) name = kernels[i].name;
  if (text_cap < text_len + 512) {
    text_cap = text_cap ? 2 * text_cap : 1 << 16;
    text = realloc(text, text_cap);
  }
  text_len += (size_t)snprintf(text + text_len, 512, "%.400s %u %u %u %u\n", name, g.x, g.y, g.z, b.x);
  return SUCCESS;
}
