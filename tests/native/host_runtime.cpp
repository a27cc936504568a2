// A stand-in for the HIP runtime, for tests of the library's host code on a machine
// without a device: device memory is host memory, copies are done at once, and kernels
// are not run but handed, with their name, grid and arguments, to a callback.  Linked
// with the host code of the library's sources by build_host.py.
#include <hip/hip_runtime_api.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

namespace {
std::map<const void*, std::string>& kernels() {  // filled while the library is loaded
  static std::map<const void*, std::string> m;
  return m;
}
struct Config {
  dim3 grid, block;
  size_t lds;
  hipStream_t stream;
};
Config g_config;
uintptr_t g_handles = 0x1000;  // streams and events: distinct values, never followed

typedef void (*launch_fn)(const char* name, unsigned gx, unsigned gy, unsigned gz, unsigned threads, size_t lds,
                          void* stream, void** args);
typedef int (*copy_fn)(void* dst, size_t bytes);
typedef float (*clock_fn)();
launch_fn g_launch = nullptr;
copy_fn g_copy = nullptr;
clock_fn g_clock = nullptr;
bool g_capturing = false;
}  // namespace

extern "C" {
// What the tests set: callbacks of launches, of copies to the device (not 0: refused) and
// of timed event pairs, and whether every stream says that it is being captured.
void host_on_launch(launch_fn f) { g_launch = f; }
void host_on_copy(copy_fn f) { g_copy = f; }
void host_on_elapsed(clock_fn f) { g_clock = f; }
void host_capturing(int on) { g_capturing = on != 0; }

void** __hipRegisterFatBinary(const void*) { return reinterpret_cast<void**>(&g_config); }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* fn, char*, const char* name, unsigned, uint3*, uint3*, dim3*, dim3*,
                           int*) {
  kernels()[fn] = name;
}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t s) {
  g_config = {grid, block, lds, s};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* s) {
  *grid = g_config.grid;
  *block = g_config.block;
  *lds = g_config.lds;
  *s = g_config.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* fn, dim3 grid, dim3 block, void** args, size_t lds, hipStream_t s) {
  if (g_launch)
    g_launch(kernels()[fn].c_str(), grid.x, grid.y, grid.z, block.x * block.y * block.z, lds, s, args);
  return hipSuccess;
}

hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind kind, hipStream_t) {
  if (kind == hipMemcpyHostToDevice && g_copy && g_copy(dst, n)) return hipErrorInvalidValue;
  memcpy(dst, src, n);
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) {
  static void* mem = calloc(1, (size_t)64 << 20);
  *p = mem;
  return hipSuccess;
}

hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { return *v = 256, hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { return *n = 2, hipSuccess; }

hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = reinterpret_cast<hipStream_t>(g_handles += 16);
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* st) {
  *st = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) {
  *e = reinterpret_cast<hipEvent_t>(g_handles += 16);
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = g_clock ? g_clock() : 1.0f;
  return hipSuccess;
}
// Solves read their state back from the device; no test here runs one.
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipErrorNotSupported; }
hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) { return hipErrorNotSupported; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
}
