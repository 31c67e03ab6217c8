/* A HIP runtime that does nothing: the library's host code runs against it without a GPU, and tests read
 * which kernels it launched and let chosen calls fail.  Loaded with global symbols before liblbrr.so.
 * Device pointers are made up and never read; pinned host memory is ordinary memory. */
#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;
enum { kOk = 0, kOutOfMemory = 2, kNotSupported = 801, kMaxKernels = 4096, kMaxLaunches = 4096 };

/* ---- what the tests set and read ---- */
int fake_fail_pool_create, fake_fail_pool_malloc, fake_capturing;
static struct { const void* host; const char* name; } kernels[kMaxKernels];
static int nkernels;
static struct { const char* name; uint32_t grid[3], block[3]; } launches[kMaxLaunches];
static int nlaunches;
static char* next_device = (char*)0x100000000000;

void fake_reset(void) { nlaunches = 0; }
int fake_launches(void) { return nlaunches; }
const char* fake_kernel(int i) { return launches[i].name; }
const uint32_t* fake_grid(int i) { return launches[i].grid; }

/* ---- the runtime ---- */
void** __hipRegisterFatBinary(const void* data) { static void* handle; (void)data; return &handle; }
void __hipUnregisterFatBinary(void** handle) { (void)handle; }
void __hipRegisterFunction(void** handle, const void* host, char* device, const char* name, unsigned limit, void* tid,
                           void* bid, void* block, void* grid, int* size) {
  (void)handle, (void)device, (void)limit, (void)tid, (void)bid, (void)block, (void)grid, (void)size;
  if (nkernels < kMaxKernels) {
    kernels[nkernels].host = host;
    kernels[nkernels++].name = name;
  }
}
void __hipRegisterVar(void** handle, void* var, char* host, char* device, int ext, size_t size, int constant, int global) {
  (void)handle, (void)var, (void)host, (void)device, (void)ext, (void)size, (void)constant, (void)global;
}
static struct { dim3_t grid, block; size_t shared; void* stream; } config;
int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t shared, void* stream) {
  config.grid = grid, config.block = block, config.shared = shared, config.stream = stream;
  return kOk;
}
int __hipPopCallConfiguration(dim3_t* grid, dim3_t* block, size_t* shared, void** stream) {
  *grid = config.grid, *block = config.block, *shared = config.shared, *stream = config.stream;
  return kOk;
}
int hipLaunchKernel(const void* host, dim3_t grid, dim3_t block, void** args, size_t shared, void* stream) {
  (void)args, (void)shared, (void)stream;
  if (nlaunches == kMaxLaunches) return kOutOfMemory;
  launches[nlaunches].name = "?";
  for (int i = 0; i < nkernels; ++i)
    if (kernels[i].host == host) launches[nlaunches].name = kernels[i].name;
  memcpy(launches[nlaunches].grid, &grid, sizeof grid);
  memcpy(launches[nlaunches++].block, &block, sizeof block);
  return kOk;
}
static int device_memory(void** p, size_t n) {
  *p = next_device;
  next_device += (n + 4095) / 4096 * 4096;
  return kOk;
}
int hipMalloc(void** p, size_t n) { return device_memory(p, n); }
int hipFree(void* p) { (void)p; return kOk; }
int hipFreeAsync(void* p, void* stream) { (void)p, (void)stream; return kOk; }
int hipHostMalloc(void** p, size_t n, unsigned flags) {
  (void)flags;
  return (*p = calloc(1, n)) ? kOk : kOutOfMemory;
}
int hipHostGetDevicePointer(void** d, void* p, unsigned flags) { (void)flags; *d = p; return kOk; }
int hipGetSymbolAddress(void** p, const void* symbol) { (void)symbol; return device_memory(p, 1 << 20); }
int hipMemPoolCreate(void** pool, const void* props) {
  (void)props;
  if (fake_fail_pool_create) return kNotSupported;
  *pool = pool;
  return kOk;
}
int hipMemPoolSetAttribute(void* pool, int attribute, void* value) { (void)pool, (void)attribute, (void)value; return kOk; }
int hipMallocFromPoolAsync(void** p, size_t n, void* pool, void* stream) {
  (void)pool, (void)stream;
  if (fake_fail_pool_malloc) return kOutOfMemory;
  return device_memory(p, n);
}
int hipMemcpyAsync(void* dst, const void* src, size_t n, int kind, void* stream) {
  (void)src, (void)stream;
  if (kind == 2) memset(dst, 0, n); /* device to host */
  return kOk;
}
int hipGetDevice(int* d) { *d = 0; return kOk; }
int hipSetDevice(int d) { (void)d; return kOk; }
int hipDeviceGetAttribute(int* v, int attribute, int d) {
  (void)attribute, (void)d;
  *v = 256; /* compute units, and yes to what is asked for */
  return kOk;
}
int hipDeviceSynchronize(void) { return kOk; }
int hipStreamSynchronize(void* stream) { (void)stream; return kOk; }
int hipStreamIsCapturing(void* stream, int* status) { (void)stream; *status = fake_capturing; return kOk; }
int hipStreamWaitEvent(void* stream, void* event, unsigned flags) { (void)stream, (void)event, (void)flags; return kOk; }
int hipEventCreateWithFlags(void** event, unsigned flags) { (void)flags; *event = event; return kOk; }
int hipEventRecord(void* event, void* stream) { (void)event, (void)stream; return kOk; }
int hipEventDestroy(void* event) { (void)event; return kOk; }
int hipGetLastError(void) { return kOk; }
const char* hipGetErrorString(int e) { return e == kOutOfMemory ? "out of memory" : "error"; }
