/* A HIP runtime without a device, for tests of the library's host code: memory is the host's, kernels do nothing, and the
 * n-th call of a chosen function fails.  Loaded before the library, whose HIP calls then bind to these. */
#include <stdlib.h>
#include <string.h>

enum { kOk = 0, kOutOfMemory = 2 };

static char fail_name[64];
static int fail_nth, calls;          /* of fail_name */
static int last_error;               /* until it is read */
static int host_mallocs, host_frees, device_pointers;   /* that succeeded */
static void* by_size[4096];          /* last hipHostMalloc of each small size */

void host_hip_fail(const char* name, int nth) {
  strncpy(fail_name, name, sizeof fail_name - 1);
  fail_nth = nth;
  calls = 0;
}
int host_hip_mallocs(void) { return host_mallocs; }
int host_hip_frees(void) { return host_frees; }
int host_hip_device_pointers(void) { return device_pointers; }
void* host_hip_of_size(size_t bytes) { return bytes < 4096 ? by_size[bytes] : 0; }

static int failing(const char* name) {
  if (strcmp(name, fail_name) != 0 || ++calls != fail_nth) return 0;
  last_error = kOutOfMemory;
  return 1;
}

int hipHostMalloc(void** p, size_t bytes, unsigned flags) {
  (void)flags;
  if (failing("hipHostMalloc")) return kOutOfMemory;
  *p = calloc(1, bytes);
  if (bytes < 4096) by_size[bytes] = *p;
  ++host_mallocs;
  return kOk;
}
int hipHostFree(void* p) { free(p); ++host_frees; return kOk; }
int hipHostGetDevicePointer(void** d, void* h, unsigned flags) {
  (void)flags;
  if (failing("hipHostGetDevicePointer")) return kOutOfMemory;
  *d = h;
  ++device_pointers;
  return kOk;
}
int hipMalloc(void** p, size_t bytes) { *p = calloc(1, bytes); return *p ? kOk : kOutOfMemory; }
int hipFree(void* p) { free(p); return kOk; }
int hipMemcpy(void* d, const void* s, size_t n, int kind) { (void)kind; memcpy(d, s, n); return kOk; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int kind, void* st) { (void)st; return hipMemcpy(d, s, n, kind); }
int hipGetDeviceCount(int* n) { *n = 1; return kOk; }
int hipSetDevice(int d) { (void)d; return kOk; }
int hipGetLastError(void) {
  const int e = last_error;
  last_error = kOk;
  return e;
}
const char* hipGetErrorString(int e) { return e ? "planted" : "no error"; }
int hipGetSymbolAddress(void** p, const void* symbol) { static char here; (void)symbol; *p = &here; return kOk; }
int hipFuncSetAttribute(const void* f, int what, int value) { (void)f; (void)what; (void)value; return kOk; }
int hipStreamCreateWithFlags(void** s, unsigned flags) { (void)flags; *s = malloc(1); return kOk; }
int hipStreamDestroy(void* s) { free(s); return kOk; }
int hipStreamSynchronize(void* s) { (void)s; return kOk; }
int hipEventCreate(void** e) { *e = malloc(1); return kOk; }
int hipEventCreateWithFlags(void** e, unsigned flags) { (void)flags; return hipEventCreate(e); }
int hipEventDestroy(void* e) { free(e); return kOk; }
int hipEventRecord(void* e, void* s) { (void)e; (void)s; return kOk; }
int hipEventQuery(void* e) { (void)e; return kOk; }
int hipEventSynchronize(void* e) { (void)e; return kOk; }
int hipEventElapsedTime(float* ms, void* a, void* b) { (void)a; (void)b; *ms = 0.0f; return kOk; }

typedef struct { unsigned x, y, z; } dim3;
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t l, void* s) { (void)g; (void)b; (void)l; (void)s; return kOk; }
int __hipPopCallConfiguration(dim3* g, dim3* b, size_t* l, void** s) { (void)g; (void)b; *l = 0; *s = 0; return kOk; }
int hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t l, void* s) {
  (void)f; (void)g; (void)b; (void)args; (void)l; (void)s;
  return kOk;
}
void** __hipRegisterFatBinary(const void* data) { static void* handle; (void)data; return &handle; }
void __hipUnregisterFatBinary(void** h) { (void)h; }
void __hipRegisterFunction(void** m, const void* f, char* df, const char* n, unsigned t, void* a, void* b, void* c, void* d, int* w) {
  (void)m; (void)f; (void)df; (void)n; (void)t; (void)a; (void)b; (void)c; (void)d; (void)w;
}
void __hipRegisterVar(void** m, void* v, char* hv, char* dv, int ext, size_t size, int constant, int global) {
  (void)m; (void)v; (void)hv; (void)dv; (void)ext; (void)size; (void)constant; (void)global;
}
