/* The HIP runtime calls of libmaclab.so without a device, for CPU tests of the
 * library's host side: launches are written to a list and run nothing, device
 * addresses are never read or written, and a call can be made to fail. Loaded
 * with RTLD_GLOBAL ahead of the library (tests/standin.py). */
#include <stdint.h>
#include <string.h>

typedef struct {
  uint32_t x, y, z;
} dim3_t;
typedef struct {
  const char* name; /* mangled kernel name; "copy" for a device copy */
  dim3_t grid, block;
  const void* arg[2]; /* first two kernel arguments (buffers in every step kernel); copy: src, dst */
} entry_t;

enum { MAX_ENTRIES = 1 << 16, MAX_KERNELS = 1024 };
static struct {
  const void* f;
  const char* name;
} kernels[MAX_KERNELS];
static int nkernels;
entry_t standin_log[MAX_ENTRIES];
int standin_count;
int standin_fail_event = -1; /* hipEventSynchronize: calls until one fails (-1: never) */
float standin_ms = 1.0f;     /* what hipEventElapsedTime reports */

static void add(const char* name, dim3_t grid, dim3_t block, const void* a, const void* b) {
  if (standin_count < MAX_ENTRIES) {
    entry_t e = {name, grid, block, {a, b}};
    standin_log[standin_count++] = e;
  }
}

void** __hipRegisterFatBinary(const void* data) {
  static void* module;
  (void)data;
  return &module;
}
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterVar(void** m, void* v, char* h, char* d, int e, size_t s, int c, int g) {
  (void)m, (void)v, (void)h, (void)d, (void)e, (void)s, (void)c, (void)g;
}
void __hipRegisterFunction(void** m, const void* f, char* d, const char* name, unsigned n, void* a, void* b, void* c,
                           void* e, int* w) {
  (void)m, (void)d, (void)n, (void)a, (void)b, (void)c, (void)e, (void)w;
  if (nkernels < MAX_KERNELS) {
    kernels[nkernels].f = f;
    kernels[nkernels++].name = name;
  }
}

static dim3_t cfg_grid, cfg_block;
static int last_error;
static size_t cfg_lds;
static void* cfg_stream;
int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t lds, void* stream) {
  cfg_grid = grid, cfg_block = block, cfg_lds = lds, cfg_stream = stream;
  return 0;
}
int __hipPopCallConfiguration(dim3_t* grid, dim3_t* block, size_t* lds, void** stream) {
  *grid = cfg_grid, *block = cfg_block, *lds = cfg_lds, *stream = cfg_stream;
  return 0;
}
int hipLaunchKernel(const void* f, dim3_t grid, dim3_t block, void** args, size_t lds, void* stream) {
  (void)lds, (void)stream;
  if ((uint64_t)grid.x * block.x >> 32 || (uint64_t)grid.y * block.y >> 32 || !grid.x || !grid.y || !grid.z)
    return last_error = 9; /* hipErrorInvalidConfiguration */
  for (int i = 0; i < nkernels; ++i)
    if (kernels[i].f == f) add(kernels[i].name, grid, block, *(const void**)args[0], *(const void**)args[1]);
  return 0;
}

int hipMemcpyAsync(void* dst, const void* src, size_t n, int kind, void* stream) {
  (void)stream;
  if (kind == 2) memset(dst, 0, n); /* to the host: zeros */
  if (kind == 3) add("copy", (dim3_t){1, 1, 1}, (dim3_t){1, 1, 1}, src, dst);
  return 0;
}
int hipMemsetAsync(void* p, int v, size_t n, void* s) { return (void)p, (void)v, (void)n, (void)s, 0; }
int hipGetDevice(int* d) { return *d = 0; }
int hipSetDevice(int d) { return (void)d, 0; }
int hipDeviceGetAttribute(int* v, int a, int d) { return (void)a, (void)d, *v = 256, 0; } /* compute units */
int hipGetSymbolAddress(void** p, const void* s) { return (void)s, *p = (void*)4096, 0; }
const char* hipGetErrorString(int e) { return e ? "failed on purpose" : "no error"; }
int hipGetLastError(void) {
  int e = last_error;
  return last_error = 0, e;
}
int hipEventCreate(void** e) { return *e = (void*)1, 0; }
int hipEventCreateWithFlags(void** e, unsigned f) { return (void)f, *e = (void*)1, 0; }
int hipEventDestroy(void* e) { return (void)e, 0; }
int hipEventRecord(void* e, void* s) { return (void)e, (void)s, 0; }
int hipEventSynchronize(void* e) {
  (void)e;
  return standin_fail_event >= 0 && standin_fail_event-- == 0;
}
int hipEventElapsedTime(float* ms, void* a, void* b) { return (void)a, (void)b, *ms = standin_ms, 0; }
int hipStreamCreateWithFlags(void** s, unsigned f) { return (void)f, *s = (void*)1, 0; }
int hipStreamDestroy(void* s) { return (void)s, 0; }
int hipStreamSynchronize(void* s) { return (void)s, 0; }
int hipStreamWaitEvent(void* s, void* e, unsigned f) { return (void)s, (void)e, (void)f, 0; }
int hipStreamBeginCapture(void* s, int m) { return (void)s, (void)m, 0; }
int hipStreamEndCapture(void* s, void** g) { return (void)s, *g = (void*)1, 0; }
int hipGraphInstantiate(void** x, void* g, void** n, char* l, size_t z) {
  return (void)g, (void)n, (void)l, (void)z, *x = (void*)1, 0;
}
int hipGraphLaunch(void* x, void* s) { return (void)x, (void)s, 0; }
int hipGraphDestroy(void* g) { return (void)g, 0; }
int hipGraphExecDestroy(void* x) { return (void)x, 0; }
