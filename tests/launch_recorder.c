/* Stands in for the HIP runtime where a test asks which kernels a call of libhiermoe would launch: loaded into the
 * global scope ahead of the library, it takes the library's runtime calls, notes every launch and runs nothing. */
#include <hip/hip_runtime_api.h>

enum { MOST = 1024, DEFAULT_LDS = 65536 };   /* dynamic LDS of a kernel that has not been granted more */

typedef struct {
  const char *name;
  uint32_t grid[3], block[3];
  uint64_t lds, granted;
} launch_t;

static struct { const void *fn; const char *name; uint64_t granted; } kernels[MOST];
static launch_t launches[MOST];
static int n_kernels, n_launches;
static struct { dim3 grid, block; size_t lds; hipStream_t stream; } pending;

static int find(const void *fn) {
  int i = 0;
  while (i < n_kernels && kernels[i].fn != fn) ++i;
  return i;
}

/* what the test asks */
int recorder_count(void) { return n_launches; }
const launch_t *recorder_launch(int i) { return &launches[i]; }
void recorder_reset(void) { n_launches = 0; }

/* what the library's launches and registrations call */
void **__hipRegisterFatBinary(const void *data) { static void *module; return &module; }
void __hipUnregisterFatBinary(void **module) {}
void __hipRegisterVar(void) {}
void __hipRegisterFunction(void **module, const void *fn, char *device_fn, const char *name) {
  if (n_kernels == MOST) return;
  kernels[n_kernels].fn = fn;
  kernels[n_kernels].name = name;
  kernels[n_kernels++].granted = DEFAULT_LDS;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream) {
  pending.grid = grid, pending.block = block, pending.lds = lds, pending.stream = stream;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *stream) {
  *grid = pending.grid, *block = pending.block, *lds = pending.lds, *stream = pending.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void *fn, dim3 grid, dim3 block, void **args, size_t lds, hipStream_t stream) {
  const int k = find(fn);
  if (k == n_kernels || n_launches == MOST) return hipErrorInvalidDeviceFunction;
  launches[n_launches++] = (launch_t){kernels[k].name, {grid.x, grid.y, grid.z}, {block.x, block.y, block.z}, lds, kernels[k].granted};
  return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void *fn, hipFuncAttribute attribute, int value) {
  const int k = find(fn);
  if (k == n_kernels || attribute != hipFuncAttributeMaxDynamicSharedMemorySize) return hipErrorInvalidValue;
  kernels[k].granted = value;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *value, hipDeviceAttribute_t attribute, int device) {   /* an MI355X */
  *value = attribute == hipDeviceAttributeMaxSharedMemoryPerMultiprocessor ? 163840 : 256;
  return hipSuccess;
}
hipError_t hipGetDevice(int *device) { *device = 0; return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipPeekAtLastError(void) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **address, const void *symbol) { *address = (void *)0x10000; return hipSuccess; }
hipError_t hipMemcpyAsync(void *to, const void *from, size_t n, hipMemcpyKind kind, hipStream_t stream) { return hipErrorNotSupported; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *blocks, const void *fn, int block, size_t lds) { *blocks = 1; return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t stream, hipStreamCaptureStatus *status) { *status = hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t stream) { return hipSuccess; }
