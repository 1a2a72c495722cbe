// The HIP runtime calls of libcnsf.so with no device behind them: addresses are handed out but
// not backed, kernels are written down instead of run.  Loaded into a process before the library
// (test_host_routes.py), it shows which kernels a call launches, which memory it takes, and
// what is left when a launch or an allocation is refused.
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {
struct Launched {
  std::string name;
  dim3 grid, block;
};
std::map<const void*, std::string> g_names;
std::vector<Launched> g_log;
std::map<uintptr_t, size_t> g_live;
uintptr_t g_next = (uintptr_t)1 << 44;
int g_cus = 256;
size_t g_free = (size_t)288 << 30;
long g_fail = -1;                  // launches until one is refused
hipError_t g_error = hipSuccess;   // what hipGetLastError returns next
double g_clock = 0.0;              // ms, moved on by every launch
std::map<std::string, double> g_cost;
dim3 g_grid, g_block;
size_t g_shared;
hipStream_t g_stream;

// k_pair of _ZN4cnsf6k_pairILi0E...
std::string plain_name(const char* mangled) {
  const char* p = std::strstr(mangled, "N4cnsf");
  if (!p) return mangled;
  char* end = nullptr;
  const long n = std::strtol(p + 6, &end, 10);
  return std::string(end, (size_t)n);
}
}  // namespace

extern "C" {

// ---- what a test sees and sets
size_t double_launches() { return g_log.size(); }
const char* double_name(size_t i) { return g_log[i].name.c_str(); }
unsigned double_block(size_t i) { return g_log[i].block.x; }
unsigned double_grid(size_t i) { return g_log[i].grid.x; }
void double_cus(int n) { g_cus = n; }
void double_forget() { g_log.clear(); }
void double_refuse(long after) { g_fail = after; }
void double_cost(const char* name, double ms) { g_cost[name] = ms; }
void double_memory(size_t bytes) { g_free = bytes; }
size_t double_held() {
  size_t n = 0;
  for (const auto& a : g_live) n += a.second;
  return n;
}

// ---- registration and launches
void** __hipRegisterFatBinary(const void*) {
  static void* none;
  return &none;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  g_names[host] = plain_name(name);
}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t s) {
  g_grid = grid;
  g_block = block;
  g_shared = shared;
  g_stream = s;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* s) {
  *grid = g_grid;
  *block = g_block;
  *shared = g_shared;
  *s = g_stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void**, size_t, hipStream_t) {
  if (g_fail >= 0 && g_fail-- == 0) return g_error = hipErrorOutOfMemory;
  const std::string& name = g_names[f];
  g_log.push_back({name, grid, block});
  g_clock += g_cost.count(name) ? g_cost[name] : 1.0;
  return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetLastError() {
  const hipError_t e = g_error;
  g_error = hipSuccess;
  return e;
}
const char* hipGetErrorString(hipError_t e) { return e == hipSuccess ? "ok" : "refused"; }

// ---- memory: device addresses are never touched, copies to the host give zeros
hipError_t hipMalloc(void** p, size_t n) {
  if (n > g_free) return g_error = hipErrorOutOfMemory;
  g_live[g_next] = n;
  g_free -= n;
  *p = (void*)g_next;
  g_next += (n + 4095) / 4096 * 4096;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  const auto it = g_live.find((uintptr_t)p);
  if (it == g_live.end()) return hipErrorInvalidValue;
  g_free += it->second;
  g_live.erase(it);
  return hipSuccess;
}
hipError_t hipMemGetInfo(size_t* f, size_t* t) {
  *f = g_free;
  *t = (size_t)288 << 30;
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  *p = std::calloc(1, n);
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipHostFree(void* p) {
  std::free(p);
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void*, size_t n, hipMemcpyKind k) {
  if (k == hipMemcpyDeviceToHost) std::memset(d, 0, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t) { return hipMemcpy(d, s, n, k); }
hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) {
  *p = (void*)g_next;
  return hipSuccess;
}

// ---- device, streams, events, graphs
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
  *v = a == hipDeviceAttributeMultiprocessorCount ? g_cus : 0;
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = (hipStream_t)(uintptr_t)16;
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* c) {
  *c = hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode*) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) {
  g_log.push_back({"capture", dim3(), dim3()});
  return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
  g_log.push_back({"captured", dim3(), dim3()});
  *g = (hipGraph_t)(uintptr_t)16;
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  *e = (hipGraphExec_t)(uintptr_t)16;
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) {
  if (g_fail >= 0 && g_fail-- == 0) return g_error = hipErrorOutOfMemory;
  g_log.push_back({"graph", dim3(), dim3()});
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) {
  *e = (hipEvent_t) new double(0.0);
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) {
  delete (double*)e;
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) {
  *(double*)e = g_clock;
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b) {
  *ms = (float)(*(double*)b - *(double*)a);
  return hipSuccess;
}

}  // extern "C"
