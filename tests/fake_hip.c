/* A HIP runtime for tests without a GPU: it runs nothing and prints what the library launches.  Built and loaded by
 * tests/test_launches_host.py in front of libnormtest.so.  A stream handle s > 16 belongs to device s >> 16. */
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3;
typedef uintptr_t stream_t;

static int current, capturing;
void fake_set(int device, int capture) { current = device; capturing = capture; }

static struct { const void* host; const char* name; } kernels[4096];
static int nkernels;
static struct { dim3 grid, block; size_t lds; stream_t stream; } config;

void** __hipRegisterFatBinary(const void* data) { static void* handle; (void)data; return &handle; }
void __hipUnregisterFatBinary(void** modules) { (void)modules; }
void __hipRegisterFunction(void** modules, const void* host, char* device, const char* name, unsigned limit, void* tid, void* bid,
                           dim3* block, dim3* grid, int* warp) {
  (void)modules; (void)device; (void)limit; (void)tid; (void)bid; (void)block; (void)grid; (void)warp;
  if (nkernels == 4096) abort();
  kernels[nkernels].host = host;
  kernels[nkernels++].name = name;
}
void __hipRegisterVar(void** modules, void* var, char* host, char* device, int ext, size_t size, int constant, int global) {
  (void)modules; (void)var; (void)host; (void)device; (void)ext; (void)size; (void)constant; (void)global;
}
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, stream_t stream) {
  config.grid = grid; config.block = block; config.lds = lds; config.stream = stream;
  return 0;
}
int __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, stream_t* stream) {
  *grid = config.grid; *block = config.block; *lds = config.lds; *stream = config.stream;
  return 0;
}
int hipLaunchKernel(const void* host, dim3 grid, dim3 block, void** args, size_t lds, stream_t stream) {
  (void)stream;
  for (int k = 0; k < nkernels; ++k)
    if (kernels[k].host == host) {
      printf("%s %u %u %zu", kernels[k].name, grid.x, block.x, lds);
      if (strstr(kernels[k].name, "k_step_end"))   /* the counter: the last of the 25 words of its last argument */
        printf(" %llx", (unsigned long long)((const uint64_t*)args[4])[24]);
      printf("\n");
      fflush(stdout);
      return 0;
    }
  return 98;   /* hipErrorInvalidDeviceFunction */
}
int hipGetDevice(int* device) { *device = current; return 0; }
int hipStreamGetDevice(stream_t stream, int* device) {
  *device = stream > 16 ? (int)(stream >> 16) : current;
  return 0;
}
int hipStreamIsCapturing(stream_t stream, int* status) { (void)stream; *status = capturing; return 0; }
int hipGetSymbolAddress(void** ptr, const void* symbol) { (void)symbol; *ptr = (void*)(uintptr_t)0x10000000; return 0; }
int hipDeviceGetAttribute(int* value, int attribute, int device) { (void)attribute; (void)device; *value = 256; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* blocks, const void* host, int threads, size_t lds) {
  (void)host; (void)threads; (void)lds;
  *blocks = 4;
  return 0;
}
int hipGetLastError(void) { return 0; }
const char* hipGetErrorString(int code) { (void)code; return "fake"; }
