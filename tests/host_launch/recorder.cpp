// Stands in for the HIP runtime calls of libcutqc.so on a machine without a
// device: kernel launches, copies and synchronisations are written down and
// succeed, except a launch that the runtime would refuse (an empty grid, or
// 2^32 threads and more in a dimension).  Loaded before the library with its
// symbols global, so the library's calls resolve here.  Host code only:
// device memory is never touched, copies back to the host read zeros.
#include <cxxabi.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "kernels.hpp"

namespace {

std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> m;
  return m;
}
std::string& log() {
  static std::string s;
  return s;
}
hipError_t g_last = hipSuccess;
struct Config {
  dim3 grid, block;
  size_t shared;
  hipStream_t stream;
};
std::vector<Config>& stack() {
  static std::vector<Config> s;
  return s;
}

void add(const std::string& event) { log() += (log().empty() ? "" : ", ") + event; }

template <typename T>
T* fake() {
  static uintptr_t next = 0x1000;
  return reinterpret_cast<T*>(next += 0x1000);
}

}  // namespace

extern "C" {

const char* recorder_events() {
  static std::string out;
  out = "[" + log() + "]";
  return out.c_str();
}
void recorder_clear() { log().clear(); }

void** __hipRegisterFatBinary(const void*) {
  static void* handle = nullptr;
  return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, dim3*, dim3*,
                           int*) {
  int status = 0;
  char* d = abi::__cxa_demangle(name, nullptr, nullptr, &status);
  std::string s = status == 0 ? d : name;
  std::free(d);
  names()[host] = s;
}

hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t stream) {
  stack().push_back(Config{grid, block, shared, stream});
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* stream) {
  const Config c = stack().back();
  stack().pop_back();
  *grid = c.grid;
  *block = c.block;
  *shared = c.shared;
  *stream = c.stream;
  return hipSuccess;
}

hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void**, size_t, hipStream_t) {
  const uint64_t gx = grid.x, gy = grid.y, gz = grid.z;
  const bool ok = gx && gy && gz && gx * block.x < (1ull << 32) && gy * block.y < (1ull << 32) &&
                  gz * block.z < (1ull << 32) && gy <= 65535 && gz <= 65535;
  char buf[256];
  std::snprintf(buf, sizeof buf, "\", \"grid\": [%u, %u, %u], \"block\": %u, \"ok\": %s}", grid.x, grid.y, grid.z,
                block.x, ok ? "true" : "false");
  add("{\"kernel\": \"" + names()[f] + buf);
  if (!ok) g_last = hipErrorInvalidConfiguration;
  return ok ? hipSuccess : hipErrorInvalidConfiguration;
}
hipError_t hipGetLastError() {
  const hipError_t e = g_last;
  g_last = hipSuccess;
  return e;
}
const char* hipGetErrorString(hipError_t) { return "recorded"; }

// The upload of a dynamic-definition batch is its device programs, one every
// 16-byte multiple of their size.
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t bytes, hipMemcpyKind kind, hipStream_t) {
  if (kind == hipMemcpyDeviceToHost) std::memset(dst, 0, bytes);
  const size_t stride = (sizeof(cq::DDProgram) + 15) / 16 * 16;
  if (kind == hipMemcpyHostToDevice && bytes % stride == 0) {
    std::string s = "{\"programs\": [";
    for (size_t at = 0; at < bytes; at += stride) {
      cq::DDProgram p;
      std::memcpy(static_cast<void*>(&p), static_cast<const char*>(src) + at, sizeof p);
      char buf[128];
      std::snprintf(buf, sizeof buf, "%s{\"prune\": %d, \"balance\": %d, \"cscale\": %d}", at ? ", " : "", p.prune,
                    p.balance, p.cscale);
      s += buf;
    }
    add(s + "]}");
  }
  return hipSuccess;
}

hipError_t hipGetDevice(int* dev) {
  *dev = 0;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* value, hipDeviceAttribute_t, int) {
  *value = 256;
  return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_t* p, int) {
  std::memset(static_cast<void*>(p), 0, sizeof *p);
  std::strcpy(p->gcnArchName, "gfx950");
  p->multiProcessorCount = 256;
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = fake<ihipStream_t>();
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
  *s = hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) {
  *e = fake<ihipEvent_t>();
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 1.0f;
  return hipSuccess;
}

}  // extern "C"
