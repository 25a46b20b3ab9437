// Stand-ins for the HIP runtime calls that libsvlf makes, so that the library's
// host code runs without a GPU: nothing is launched, the calls are recorded.
// Linked with the library's own objects in place of the HIP runtime.
#include <hip/hip_runtime.h>

#include <cstring>
#include <map>
#include <string>

#include "svlf_internal.hpp"

namespace {

struct Config {
  dim3 grid, block;
  size_t lds;
  hipStream_t stream;
};
Config g_config;
std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> m;
  return m;
}
std::map<const void*, int> g_lds_limit;
// what the calls since the last rec_reset() did
struct {
  int launches, traces, live_traces, live_counts, lds_limit_changes;
  uint64_t live_begin, live_end;      // addresses of the live-ray arrays of the last live trace
} g_rec;

}  // namespace

extern "C" {

void rec_reset() { std::memset(&g_rec, 0, sizeof(g_rec)); }
int rec_launches() { return g_rec.launches; }
int rec_traces() { return g_rec.traces; }
int rec_live_traces() { return g_rec.live_traces; }
int rec_live_counts() { return g_rec.live_counts; }
int rec_lds_limit_changes() { return g_rec.lds_limit_changes; }
uint64_t rec_live_begin() { return g_rec.live_begin; }
uint64_t rec_live_end() { return g_rec.live_end; }
int rec_dealt_items(int n_items, int blocks) { return svlf::dealt_items(n_items, blocks); }

void** __hipRegisterFatBinary(const void*) {
  static void* handle;
  return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, uint3*, uint3*, dim3*, dim3*,
                           int*) {
  names()[host] = name;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream) {
  g_config = {grid, block, lds, stream};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* stream) {
  *grid = g_config.grid;
  *block = g_config.block;
  *lds = g_config.lds;
  *stream = g_config.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void** args, size_t, hipStream_t) {
  ++g_rec.launches;
  const bool trace = names()[f].find("k_trace_internal") != std::string::npos;
  const bool count = names()[f].find("k_live") != std::string::npos;
  g_rec.traces += trace;
  g_rec.live_counts += count;
  if (trace || count) {
    const auto& tab = *static_cast<const svlf::SceneTable*>(args[0]);
    if (tab.live_n != nullptr) {
      g_rec.live_traces += trace;
      g_rec.live_begin = reinterpret_cast<uint64_t>(tab.live_n);
      g_rec.live_end = reinterpret_cast<uint64_t>(tab.live_mask + tab.n_trace);
    }
  }
  return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void* f, hipFuncAttribute, int value) {
  const auto it = g_lds_limit.find(f);
  if (it != g_lds_limit.end() && it->second != value) ++g_rec.lds_limit_changes;
  g_lds_limit[f] = value;
  return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
  *n = 2;
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
  *v = 256;
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "no HIP runtime"; }
hipError_t hipEventCreateWithFlags(hipEvent_t*, unsigned) { return hipErrorNotSupported; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipStreamCreateWithFlags(hipStream_t*, unsigned) { return hipErrorNotSupported; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipErrorNotSupported; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipErrorNotSupported; }
hipError_t hipGetSymbolAddress(void**, const void*) { return hipErrorNotSupported; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipErrorNotSupported; }
int roctxRangePushA(const char*) { return 0; }
int roctxRangePop() { return 0; }

}  // extern "C"
