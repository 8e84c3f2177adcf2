/* A stand-in for the HIP runtime: device memory is host memory, launches are only noted by name, and a chosen allocation
 * fails.  Loaded into the global scope before libfpsched.so, it shows on a machine without a GPU which kernels a call
 * launches and what the library does when the runtime refuses something. */
#define __HIP_PLATFORM_AMD__
#include <hip/hip_runtime_api.h>
#include <stdlib.h>
#include <string.h>

enum { kMost = 4096 };
static struct { const void* host; const char* name; } kernels[kMost];
static const char* launches[kMost];
static struct { unsigned grid, block, lds, word; } shapes[kMost];
static int n_kernels, n_launches, mallocs_to_failure;
static hipError_t last_error;

/* the nth allocation from now on fails (0: none); returns how many were left to the one asked for before */
int stub_fail_malloc(int nth) {
  const int left = mallocs_to_failure;
  mallocs_to_failure = nth;
  return left;
}
void stub_reset(void) { n_launches = 0; }
int stub_launches(void) { return n_launches; }
const char* stub_launched(int i) { return launches[i]; }
unsigned stub_grid(int i) { return shapes[i].grid; }
unsigned stub_block(int i) { return shapes[i].block; }
unsigned stub_lds(int i) { return shapes[i].lds; }
/* of launches of kernels with this in their names, the first four bytes of an argument */
static const char* watched_kernel;
static int watched_argument;
void stub_watch(const char* kernel, int argument) { watched_kernel = kernel; watched_argument = argument; }
unsigned stub_word(int i) { return shapes[i].word; }

static hipError_t note(hipError_t e) {
  if (e != hipSuccess) last_error = e;
  return e;
}
hipError_t hipGetLastError(void) {
  const hipError_t e = last_error;
  last_error = hipSuccess;
  return e;
}
hipError_t hipMalloc(void** p, size_t n) {
  if (mallocs_to_failure > 0 && --mallocs_to_failure == 0) return note(hipErrorOutOfMemory);
  *p = malloc(n);
  return hipSuccess;
}
hipError_t hipFree(void* p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void* to, const void* from, size_t n, hipMemcpyKind kind) {
  (void)kind;
  if (!to || !from) return note(hipErrorInvalidValue);
  memcpy(to, from, n);
  return hipSuccess;
}
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int d) { (void)d; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void* f, hipFuncAttribute a, int v) { (void)f; (void)a; (void)v; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int d) {
  (void)d;
  *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 160 * 1024;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void* symbol) { *p = (void*)symbol; return hipSuccess; }

void** __hipRegisterFatBinary(const void* data) { static void* module; (void)data; return &module; }
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterVar(void** m, void* var, char* host, char* device, int ext, size_t size, int constant, int global) {
  (void)m; (void)var; (void)host; (void)device; (void)ext; (void)size; (void)constant; (void)global;
}
void __hipRegisterFunction(void** m, const void* host, char* device, const char* name, unsigned limit, void* tid, void* bid,
                           dim3* block, dim3* grid, int* wave) {
  (void)m; (void)device; (void)limit; (void)tid; (void)bid; (void)block; (void)grid; (void)wave;
  if (n_kernels < kMost) { kernels[n_kernels].host = host; kernels[n_kernels++].name = name; }
}
static struct { dim3 grid, block; size_t lds; hipStream_t stream; } call;
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream) {
  call.grid = grid; call.block = block; call.lds = lds; call.stream = stream;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* stream) {
  *grid = call.grid; *block = call.block; *lds = call.lds; *stream = call.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* host, dim3 grid, dim3 block, void** args, size_t lds, hipStream_t stream) {
  (void)stream;
  for (int i = 0; i < n_kernels; ++i)
    if (kernels[i].host == host && n_launches < kMost) {
      shapes[n_launches].grid = grid.x;
      shapes[n_launches].block = block.x;
      shapes[n_launches].lds = (unsigned)lds;
      shapes[n_launches].word = 0;
      if (watched_kernel && strstr(kernels[i].name, watched_kernel)) memcpy(&shapes[n_launches].word, args[watched_argument], 4);
      launches[n_launches++] = kernels[i].name;
    }
  return note(hipSuccess);
}
