// A stand-in for the HIP runtime that runs nothing and records every kernel
// launch (kernel name, grid, block, host thread), so that tests can see on the
// CPU which kernels a call of the library launches, in which order.
//
// It reports one GPU of 256 CUs and 160 KB of LDS.  Between two launches of
// the same thread it can pause (recorder_pause_us), so that other threads'
// launches come in between wherever nothing keeps them out, and it can refuse
// the launches of a kernel (recorder_fail).
#include <hip/hip_runtime_api.h>

#include <cxxabi.h>
#include <unistd.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <thread>
#include <vector>

namespace {
struct Launch {
  std::string kernel;
  unsigned grid, block;
  size_t thread;
};
std::mutex mu;
std::map<const void*, std::string> kernels;
std::vector<Launch> launches;
std::string refused;
int pause_us = 0;

struct Config {
  dim3 grid, block;
  size_t shared;
  hipStream_t stream;
};
thread_local Config config;
thread_local hipError_t last = hipSuccess;
char device_word[256] __attribute__((aligned(256)));
}  // namespace

extern "C" {

void** __hipRegisterFatBinary(const void*) {
  static void* module = nullptr;
  return &module;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*,
                           void*, void*, void*, int*) {
  int st = 0;
  char* plain = abi::__cxa_demangle(name, nullptr, nullptr, &st);
  std::lock_guard<std::mutex> lk(mu);
  kernels[host] = plain ? plain : name;
  std::free(plain);
}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t stream) {
  config = {grid, block, shared, stream};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* stream) {
  *grid = config.grid;
  *block = config.block;
  *shared = config.shared;
  *stream = config.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void**, size_t, hipStream_t) {
  {
    std::lock_guard<std::mutex> lk(mu);
    const std::string& name = kernels[f];
    if (!refused.empty() && name.find(refused) != std::string::npos) {
      last = hipErrorLaunchFailure;
      return last;
    }
    launches.push_back({name, grid.x, block.x,
                        std::hash<std::thread::id>()(std::this_thread::get_id())});
  }
  if (pause_us > 0) usleep(pause_us);
  return hipSuccess;
}
hipError_t hipGetLastError() {
  const hipError_t e = last;
  last = hipSuccess;
  return e;
}
hipError_t hipGetDevice(int* dev) {
  *dev = 0;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  std::memset(p, 0, sizeof(*p));
  p->multiProcessorCount = 256;
  p->maxSharedMemoryPerMultiProcessor = 160 << 10;
  return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
  *n = 1;
  return hipSuccess;
}
hipError_t hipFuncGetAttributes(hipFuncAttributes* a, const void*) {
  std::memset(a, 0, sizeof(*a));
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) {
  *p = device_word;   // an address for launches that never run
  return hipSuccess;
}
hipError_t hipMemcpy(void*, const void*, size_t, hipMemcpyKind) { return hipErrorNoDevice; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }

int recorder_count() {
  std::lock_guard<std::mutex> lk(mu);
  return (int)launches.size();
}
void recorder_clear() {
  std::lock_guard<std::mutex> lk(mu);
  launches.clear();
}
void recorder_get(int i, char* name, int n, unsigned* grid, unsigned* block, size_t* thread) {
  std::lock_guard<std::mutex> lk(mu);
  const Launch& l = launches[i];
  std::strncpy(name, l.kernel.c_str(), n - 1);
  name[n - 1] = 0;
  *grid = l.grid;
  *block = l.block;
  *thread = l.thread;
}
void recorder_pause_us(int us) { pause_us = us; }
void recorder_fail(const char* kernel) {
  std::lock_guard<std::mutex> lk(mu);
  refused = kernel;
}
}
