/* The HIP runtime calls the library makes, on host memory: nothing is launched, every call is written to a
 * log.  Loaded before the library (RTLD_GLOBAL), it lets the tests follow the host path, with failures a GPU
 * run cannot bring about, where there is no GPU.  Device memory is zeroed host memory, so every kernel's
 * result reads as zero. */
#include <hip/hip_runtime_api.h>
#include <stdarg.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

static char log_text[1 << 22];
static size_t log_used;
static int fail_host_mallocs; /* pinned allocations still to fail */
static int fail_copies;       /* asynchronous copies still to fail */
static size_t fail_malloc_of; /* device allocations of this size fail */
static uintptr_t next_handle = 0x1000;

static void note(const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  if (log_used + 512 < sizeof(log_text)) log_used += vsnprintf(log_text + log_used, 512, fmt, ap);
  va_end(ap);
}
const char* fake_log(void) { return log_text; }
void fake_clear(void) { log_used = 0, log_text[0] = 0; }
void fake_fail_host_mallocs(int n) { fail_host_mallocs = n; }
void fake_fail_copies(int n) { fail_copies = n; }
void fake_fail_malloc_of(size_t n) { fail_malloc_of = n; }

/* kernels by the address of their host stub */
static struct { const void* stub; char name[160]; } kernels[4096];
static int n_kernels;
static hipModule_t module;
hipModule_t* __hipRegisterFatBinary(const void* data) { (void)data; return &module; }
void __hipUnregisterFatBinary(hipModule_t* m) { (void)m; }
void __hipRegisterVar(void* m, void* v, char* h, char* d, int e, size_t s, int c, int g) {
  (void)m, (void)v, (void)h, (void)d, (void)e, (void)s, (void)c, (void)g;
}
void __hipRegisterFunction(hipModule_t* m, const void* stub, char* dev, const char* name, unsigned lim, uint3* t,
                           uint3* b, dim3* bd, dim3* gd, int* w) {
  (void)m, (void)dev, (void)lim, (void)t, (void)b, (void)bd, (void)gd, (void)w;
  if (n_kernels < 4096) {
    kernels[n_kernels].stub = stub;
    snprintf(kernels[n_kernels++].name, 160, "%s", name);
  }
}
static struct { dim3 g, b; size_t shm; hipStream_t s; } config;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t shm, hipStream_t s) {
  config.g = g, config.b = b, config.shm = shm, config.s = s;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* shm, hipStream_t* s) {
  *g = config.g, *b = config.b, *shm = config.shm, *s = config.s;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* stub, dim3 g, dim3 b, void** args, size_t shm, hipStream_t s) {
  const char* name = "?";
  for (int k = 0; k < n_kernels; ++k)
    if (kernels[k].stub == stub) name = kernels[k].name;
  (void)b, (void)shm;
  note("launch %p %s %u %u", (void*)s, name, g.x, g.y);
  if (strstr(name, "publish_kernel")) note(" dst %p", *(void**)args[1]);
  note("\n");
  return hipSuccess;
}

hipError_t hipMalloc(void** p, size_t n) {
  note("malloc %zu\n", n);
  if (n == fail_malloc_of) {
    *p = NULL;
    return hipErrorOutOfMemory;
  }
  return (*p = calloc(1, n + 256)) ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void* p) { free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned flags) {
  (void)flags;
  note("hostmalloc %zu%s\n", n, fail_host_mallocs ? " fails" : "");
  if (fail_host_mallocs) {
    --fail_host_mallocs;
    *p = NULL;
    return hipErrorOutOfMemory;
  }
  return (*p = calloc(1, n)) ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipHostFree(void* p) { note("hostfree\n"); free(p); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind k) { (void)k; memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t st) {
  (void)k;
  if (fail_copies) {
    --fail_copies;
    return hipErrorInvalidValue;
  }
  double first = 0;
  if (n >= sizeof(first)) memcpy(&first, s, sizeof(first));
  note("copy %p %zu first %.17g\n", (void*)st, n, first);
  memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemset(void* d, int v, size_t n) { memset(d, v, n); return hipSuccess; }
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t s) { (void)s; memset(d, v, n); return hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
  (void)p;
  memset(a, 0, sizeof(*a));
  return hipErrorInvalidValue;
}
hipError_t hipGetSymbolAddress(void** p, const void* s) { (void)s; *p = NULL; return hipErrorInvalidValue; }

hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int d) {
  (void)d;
  memset(p, 0, sizeof(*p));
  strcpy(p->gcnArchName, "gfx950");
  p->multiProcessorCount = 256;
  return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
const char* hipGetErrorString(hipError_t e) { (void)e; return "fake"; }

static hipError_t handle(void** h) { *h = (void*)(next_handle += 0x10); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { return handle((void**)e); }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned f) { (void)f; return handle((void**)e); }
hipError_t hipEventDestroy(hipEvent_t e) { (void)e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { (void)e, (void)s; return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t e) { (void)e; return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b) { (void)a, (void)b; *ms = 1.f; return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned f) { (void)f; return handle((void**)s); }
hipError_t hipStreamDestroy(hipStream_t s) { (void)s; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { note("sync %p\n", (void*)s); return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned f) { (void)s, (void)e, (void)f; return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode m) { (void)s, (void)m; return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t* g) { (void)s; return handle((void**)g); }
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t g, hipGraphNode_t* n, char* b, size_t z) {
  (void)g, (void)n, (void)b, (void)z;
  return handle((void**)e);
}
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t s) { (void)e; note("graph %p\n", (void*)s); return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t g) { (void)g; return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t e) { (void)e; return hipSuccess; }
