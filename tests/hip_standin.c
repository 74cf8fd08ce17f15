/* A stand-in for the HIP host calls that the library makes, for CPU tests of
 * its host code: preloaded into a process without a GPU, it hands out host
 * memory, copies at once, runs no kernel and writes down what is called, and
 * the test says which launch fails and how often the stream is still busy.
 *
 * The log holds one word per call: a launch as the kernel's mangled name and
 * its grid ("_ZN2lc...:40"), "copy", "sync" and "query". */
#include <hip/hip_runtime_api.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#define MAX_RANGES 65536
#define MAX_KERNELS 1024
#define LOG_BYTES (1 << 20)

static struct { char *base; size_t size; hipMemoryType type; } ranges[MAX_RANGES];
static int n_ranges;
static struct { const void *host; const char *name; } kernels[MAX_KERNELS];
static int n_kernels;
static char log_text[LOG_BYTES];
static size_t log_len;
static int fail_launch, busy_queries;
static hipError_t last_error;
static dim3 cfg_grid, cfg_block;
static size_t cfg_lds;
static hipStream_t cfg_stream;

/* ---- the test's side --------------------------------------------------------- */
const char *standin_log(void) { return log_text; }
void standin_clear(void) { log_len = 0; log_text[0] = 0; }
void standin_fail_launch(int n) { fail_launch = n; }   /* the n-th launch from now on; 0: none */
void standin_busy(int n) { busy_queries = n; }         /* so many queries say "not ready" */
void standin_stale_error(void) { last_error = hipErrorOutOfMemory; } /* as an earlier call of the program leaves it */
void *standin_alloc(size_t bytes, int type) {
  void *p = aligned_alloc(256, (bytes + 255) / 256 * 256);
  if (!p || n_ranges == MAX_RANGES) abort();
  memset(p, 0, bytes);
  ranges[n_ranges].base = p;
  ranges[n_ranges].size = bytes;
  ranges[n_ranges++].type = (hipMemoryType)type;
  return p;
}

static void note(const char *what) {
  const size_t n = strlen(what);
  if (log_len + n + 2 > LOG_BYTES) abort();
  memcpy(log_text + log_len, what, n);
  log_len += n;
  log_text[log_len++] = ' ';
  log_text[log_len] = 0;
}

static int find(const void *p) {
  for (int i = n_ranges - 1; i >= 0; --i)
    if ((const char *)p >= ranges[i].base && (const char *)p < ranges[i].base + ranges[i].size) return i;
  return -1;
}

static hipError_t drop(void *p) {
  const int i = p ? find(p) : -1;
  if (i >= 0 && ranges[i].base == p) ranges[i] = ranges[--n_ranges];
  free(p);
  return hipSuccess;
}

/* ---- modules and launches ------------------------------------------------------ */
void **__hipRegisterFatBinary(const void *data) { (void)data; static void *module; return &module; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterFunction(void **m, const void *host, char *device, const char *name, unsigned int limit, void *tid,
                           void *bid, dim3 *block, dim3 *grid, int *warp) {
  (void)m; (void)device; (void)limit; (void)tid; (void)bid; (void)block; (void)grid; (void)warp;
  if (n_kernels == MAX_KERNELS) abort();
  kernels[n_kernels].host = host;
  kernels[n_kernels++].name = name;
}
void __hipRegisterVar(void **m, void *var, char *host, char *name, int ext, size_t size, int constant, int global) {
  (void)m; (void)var; (void)host; (void)name; (void)ext; (void)size; (void)constant; (void)global;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t s) {
  cfg_grid = grid; cfg_block = block; cfg_lds = lds; cfg_stream = s;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *s) {
  *grid = cfg_grid; *block = cfg_block; *lds = cfg_lds; *s = cfg_stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t lds, hipStream_t s) {
  (void)block; (void)args; (void)lds; (void)s;
  char text[512];
  const char *name = "?";
  for (int i = 0; i < n_kernels; ++i)
    if (kernels[i].host == f) name = kernels[i].name;
  snprintf(text, sizeof text, "%s:%u", name, grid.x);
  note(text);
  if (fail_launch && --fail_launch == 0) return last_error = hipErrorLaunchFailure;
  return hipSuccess;
}

/* ---- memory -------------------------------------------------------------------- */
hipError_t hipMalloc(void **p, size_t n) { *p = standin_alloc(n, hipMemoryTypeDevice); return hipSuccess; }
hipError_t hipFree(void *p) { return drop(p); }
hipError_t hipHostMalloc(void **p, size_t n, unsigned int flags) {
  (void)flags;
  *p = standin_alloc(n, hipMemoryTypeHost);
  return hipSuccess;
}
hipError_t hipHostFree(void *p) { return drop(p); }
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned int flags) { (void)flags; *d = h; return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t st) {
  (void)k; (void)st;
  note("copy");
  memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p) {
  const int i = find(p);
  memset(a, 0, sizeof *a);
  if (i < 0) return last_error = hipErrorInvalidValue;
  a->type = ranges[i].type;
  a->devicePointer = (void *)p;
  a->hostPointer = ranges[i].type == hipMemoryTypeHost ? (void *)p : NULL;
  return hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t *base, size_t *size, hipDeviceptr_t p) {
  const int i = find(p);
  if (i < 0) return last_error = hipErrorNotFound;
  *base = ranges[i].base;
  *size = ranges[i].size;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *sym) { (void)p; (void)sym; return last_error = hipErrorInvalidSymbol; }

/* ---- device, stream, events ------------------------------------------------------ */
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int d) { (void)d; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int d) { (void)a; (void)d; *v = 160 << 10; return hipSuccess; }
hipError_t hipGetLastError(void) {
  const hipError_t e = last_error;
  last_error = hipSuccess;
  return e;
}
const char *hipGetErrorString(hipError_t e) { return e == hipSuccess ? "no error" : "stand-in error"; }
hipError_t hipStreamSynchronize(hipStream_t s) { (void)s; note("sync"); return hipSuccess; }
hipError_t hipStreamQuery(hipStream_t s) {
  (void)s;
  note("query");
  if (busy_queries > 0) {
    --busy_queries;
    return hipErrorNotReady;
  }
  return hipSuccess;
}
