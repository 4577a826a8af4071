// A device of a few counters in place of the HIP runtime, for host checks of
// what the library asks of it: link a check that includes this header with
// libatlas_nabla.so, and the functions here take the runtime's place.  Memory
// is addresses only (never touched), kernels are names that are noted down.
#pragma once
#include <cxxabi.h>
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <set>
#include <string>
#include <vector>

struct FakeDevice {
  // memory
  size_t total = size_t(288) << 30;    // bytes the device says it has
  size_t limit = SIZE_MAX, live = 0;   // bytes it has left to give, and holds
  int mallocs = 0, refused = 0;
  std::map<uintptr_t, size_t> blocks;
  uintptr_t next = uintptr_t(1) << 40;
  // streams being captured: `here` by this thread, `elsewhere` by another one
  std::set<hipStream_t> here;
  bool elsewhere = false;
  int broken = 0;                      // calls that would have broken a capture
  hipStreamCaptureMode mode = hipStreamCaptureModeGlobal;
  // kernels
  std::map<const void*, std::string> names;
  std::vector<std::string> launches;
  std::vector<int> orders;             // of the k_tile launches: their `remap` argument
  hipError_t last = hipSuccess;
  int stream_count = 0;

  static FakeDevice& get() {
    static FakeDevice* d = new FakeDevice;   // registrations come before main
    return *d;
  }
  // A call that no capture allows (memory, waiting for the device).
  bool unsafe() {
    if ((here.empty() && !elsewhere) || mode == hipStreamCaptureModeRelaxed) return false;
    ++broken;
    return true;
  }
  hipError_t set(hipError_t e) {
    if (e != hipSuccess) last = e;
    return e;
  }
  // "k_tile<float, 1, 0>" of the kernel's full name
  static std::string short_name(const std::string& s) {
    size_t a = s.find("k_");
    return a == std::string::npos ? s : s.substr(a, s.find('(', a) - a);
  }
  int count(const char* prefix) const {
    int n = 0;
    for (const auto& s : launches) n += s.rfind(prefix, 0) == 0;
    return n;
  }
};

inline FakeDevice& dev() { return FakeDevice::get(); }

extern "C" {
void** __hipRegisterFatBinary(const void*) {
  static void* handle[1] = {};
  return handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*,
                           int*) {
  int st = 0;
  char* d = abi::__cxa_demangle(name, nullptr, nullptr, &st);
  std::string s = st == 0 ? d : name;
  free(d);
  // "(anonymous namespace)" has a bracket of its own
  const size_t p = s.find("(anonymous namespace)::");
  if (p != std::string::npos) s.erase(p, 23);
  dev().names[host] = FakeDevice::short_name(s);
}
static dim3 fake_grid, fake_block;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t, hipStream_t) {
  fake_grid = g;
  fake_block = b;
  return hipSuccess;
}
static hipStream_t fake_stream;
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* s, hipStream_t* st) {
  *g = fake_grid;
  *b = fake_block;
  *s = 0;
  *st = fake_stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void** args, size_t, hipStream_t) {
  dev().launches.push_back(dev().names.count(f) ? dev().names[f] : "?");
  if (dev().launches.back().rfind("k_tile<", 0) == 0) dev().orders.push_back(*static_cast<int*>(args[2]));
  return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
  *n = 1;
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceCount(int* n) {
  *n = 1;
  return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  p->multiProcessorCount = 256;
  p->totalGlobalMem = dev().total;
  return hipSuccess;
}
const char* hipGetErrorString(hipError_t e) {
  return e == hipErrorOutOfMemory ? "out of memory" : e == hipErrorStreamCaptureUnsupported ? "stream capture" : "error";
}
hipError_t hipGetLastError() {
  const hipError_t e = dev().last;
  dev().last = hipSuccess;
  return e;
}
hipError_t hipMalloc(void** p, size_t n) {
  FakeDevice& d = dev();
  ++d.mallocs;
  if (d.unsafe()) return d.set(hipErrorStreamCaptureUnsupported);
  if (n > d.limit || d.live > d.limit - n) {
    ++d.refused;
    return d.set(hipErrorOutOfMemory);
  }
  *p = reinterpret_cast<void*>(d.next);
  d.blocks[d.next] = n;
  d.live += n;
  d.next += (n + 4095) / 4096 * 4096;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  FakeDevice& d = dev();
  if (d.unsafe()) return d.set(hipErrorStreamCaptureUnsupported);
  auto it = d.blocks.find(reinterpret_cast<uintptr_t>(p));
  if (it == d.blocks.end()) {
    std::printf("FAILED: freed what is not there\n");
    std::exit(1);
  }
  d.live -= it->second;
  d.blocks.erase(it);
  return hipSuccess;
}
hipError_t hipMemcpy(void*, const void*, size_t, hipMemcpyKind) {
  return dev().unsafe() ? dev().set(hipErrorStreamCaptureUnsupported) : hipSuccess;
}
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipMemset(void*, int, size_t) {
  return dev().unsafe() ? dev().set(hipErrorStreamCaptureUnsupported) : hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st) {
  *st = dev().here.count(s) ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* m) {
  std::swap(*m, dev().mode);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
  if (!dev().here.count(s)) return hipSuccess;
  ++dev().broken;
  return dev().set(hipErrorStreamCaptureUnsupported);
}
hipError_t hipDeviceSynchronize() { return dev().unsafe() ? dev().set(hipErrorStreamCaptureUnsupported) : hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = reinterpret_cast<hipStream_t>((uintptr_t)(0x1000 + ++dev().stream_count));
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) {
  dev().here.insert(s);
  return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t* g) {
  dev().here.erase(s);
  *g = reinterpret_cast<hipGraph_t>(uintptr_t(0x2000));
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  *e = reinterpret_cast<hipGraphExec_t>(uintptr_t(0x3000));
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) {
  *p = reinterpret_cast<void*>(uintptr_t(1) << 39);
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) {
  *e = reinterpret_cast<hipEvent_t>(uintptr_t(0x4000));
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 1.0f;
  return hipSuccess;
}
}
