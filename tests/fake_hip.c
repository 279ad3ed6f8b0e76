/* A stand-in for the HIP runtime with two devices and no GPU, for tests of the library's
 * host code on the CPU.  Memory is ordinary, zeroed memory, copies are done at once, kernels
 * are not run.  What matters to a test goes to stdout, a line a call. */
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3;

static int device;
static struct { const void* host; const char* name; } kernels[256];
static int n_kernels;

int hipGetDevice(int* d) { *d = device; return 0; }
int hipSetDevice(int d) { device = d; return 0; }
int hipDeviceGetAttribute(int* v, int what, int d) { *v = 256; return 0; }
int hipDeviceGetDefaultMemPool(void** p, int d) { *p = NULL; return 0; }
int hipMemPoolSetAttribute(void* p, int what, void* v) { return 0; }
int hipGetLastError(void) { return 0; }
int hipGetSymbolAddress(void** p, const void* symbol) { *p = (void*)symbol; return 0; }
int hipMemcpyToSymbol(const void* symbol, const void* from, size_t size, size_t at, int kind) { return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int block, size_t lds) { *n = 7; return 0; }

int hipMalloc(void** p, size_t size) { *p = calloc(1, size); return 0; }
int hipFree(void* p) { free(p); return 0; }
int hipMallocAsync(void** p, size_t size, void* stream) {
  printf("device block %d %zu\n", device, size);
  *p = calloc(1, size);
  return 0;
}
int hipFreeAsync(void* p, void* stream) { free(p); return 0; }
int hipHostMalloc(void** p, size_t size, unsigned flags) {
  *p = calloc(1, size);
  printf("host block %d %u %p %zu\n", device, flags, *p, size);
  return 0;
}
int hipHostFree(void* p) { free(p); return 0; }
int hipMemcpyAsync(void* to, const void* from, size_t size, int kind, void* stream) {
  printf("copy %d %d %p %zu\n", device, kind, to, size);
  memcpy(to, from, size);
  return 0;
}
int hipMemsetAsync(void* p, int v, size_t size, void* stream) { memset(p, v, size); return 0; }

int hipStreamCreateWithFlags(void** s, unsigned flags) { *s = malloc(1); return 0; }
int hipStreamDestroy(void* s) { free(s); return 0; }
int hipStreamSynchronize(void* s) { return 0; }
int hipStreamWaitEvent(void* s, void* e, unsigned flags) { return 0; }
int hipEventCreateWithFlags(void** e, unsigned flags) { *e = malloc(1); return 0; }
int hipEventDestroy(void* e) { free(e); return 0; }
int hipEventRecord(void* e, void* s) { return 0; }

void** __hipRegisterFatBinary(const void* data) { static void* module; return &module; }
void __hipUnregisterFatBinary(void** m) {}
void __hipRegisterVar(void** m, void* var, char* host, char* dev, int ext, size_t size, int constant, int global) {}
void __hipRegisterFunction(void** m, const void* host, char* dev, const char* name, unsigned limit, void* a, void* b,
                           void* c, void* d, int* e) {
  kernels[n_kernels].host = host;
  kernels[n_kernels++].name = name;
}

static dim3 c_grid, c_block;
static size_t c_lds;
static void* c_stream;
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void* stream) {
  c_grid = grid, c_block = block, c_lds = lds, c_stream = stream;
  return 0;
}
int __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, void** stream) {
  *grid = c_grid, *block = c_block, *lds = c_lds, *stream = c_stream;
  return 0;
}
int hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t lds, void* stream) {
  for (int i = 0; i < n_kernels; ++i) {
    if (kernels[i].host != f) continue;
    printf("launch %d %s %u\n", device, kernels[i].name, grid.x);
    /* the counts of histogram words: the fifth argument of the one, the second of the other */
    const int at = strstr(kernels[i].name, "k_batch_stage") ? 4 : strstr(kernels[i].name, "k_batch_collect") ? 1 : -1;
    if (at >= 0) printf("words %llu\n", *(unsigned long long*)args[at]);
  }
  return 0;
}
