// The HIP runtime calls of libxeng.so without a GPU, for CPU tests of its host
// code: memory is counted but not there, kernels are not run, launches past
// the limits of the hardware packet are refused.  Loaded before libxeng.so
// with global symbols, it answers in place of the HIP runtime.
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstring>
#include <map>

static std::map<uintptr_t, size_t> g_blocks;
static uintptr_t g_next = (uintptr_t)1 << 40;
static size_t g_used = 0, g_limit = SIZE_MAX;
static hipError_t g_last = hipSuccess;
static dim3 g_grid, g_block;
static int g_timed = 0, g_fast = -1;
static int g_dummy;

static hipError_t result(hipError_t e) {
  if (e != hipSuccess) g_last = e;
  return e;
}

extern "C" {
size_t stub_used() { return g_used; }
void stub_limit(size_t bytes) { g_limit = bytes; }
// the timing after `later` others is the shortest of all from here
void stub_fast(int later) { g_timed = 0, g_fast = later; }

void** __hipRegisterFatBinary(const void*) { return reinterpret_cast<void**>(&g_dummy); }
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
void __hipUnregisterFatBinary(void**) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t, hipStream_t) {
  g_grid = grid, g_block = block;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* s) {
  *grid = g_grid, *block = g_block, *lds = 0, *s = nullptr;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void*, dim3 grid, dim3 block, void**, size_t, hipStream_t) {
  const bool fits = (uint64_t)grid.x * block.x <= UINT32_MAX && (uint64_t)grid.y * block.y <= UINT32_MAX;
  return result(fits && grid.x && grid.y ? hipSuccess : hipErrorInvalidConfiguration);
}
hipError_t hipGetLastError() {
  const hipError_t e = g_last;
  g_last = hipSuccess;
  return e;
}
const char* hipGetErrorString(hipError_t e) { return e == hipErrorInvalidConfiguration ? "invalid configuration" : "error"; }

hipError_t hipMalloc(void** p, size_t n) {
  if (n > g_limit || g_used > g_limit - n) return result(hipErrorOutOfMemory);
  *p = reinterpret_cast<void*>(g_next);
  g_blocks[g_next] = n;
  g_next += (n + 4095) / 4096 * 4096 + 4096;
  g_used += n;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  if (!p) return hipSuccess;
  auto it = g_blocks.find(reinterpret_cast<uintptr_t>(p));
  if (it == g_blocks.end()) return result(hipErrorInvalidValue);
  g_used -= it->second;
  g_blocks.erase(it);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void*) {
  std::memset(a, 0, sizeof *a);
  a->type = hipMemoryTypeDevice;
  return hipSuccess;
}

hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { return *v = 256, hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  std::memset(p, 0, sizeof *p);
  std::strcpy(p->gcnArchName, "gfx950:sramecc+:xnack-");
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { return *s = reinterpret_cast<hipStream_t>(&g_dummy), hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { return *e = reinterpret_cast<hipEvent_t>(&g_dummy), hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { return *ms = g_timed++ == g_fast ? 0.5f : 1.0f, hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) { return *g = reinterpret_cast<hipGraph_t>(&g_dummy), hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  return *e = reinterpret_cast<hipGraphExec_t>(&g_dummy), hipSuccess;
}
hipError_t hipGraphExecUpdate(hipGraphExec_t, hipGraph_t, hipGraphNode_t*, hipGraphExecUpdateResult* r) {
  return *r = hipGraphExecUpdateSuccess, hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
}
