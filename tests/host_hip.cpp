// A HIP runtime that records instead of running: the host side of the library
// (checks, allocations, launches and their arguments) can be followed on a
// machine without a GPU.  Loaded with global symbols before libptycho.so, it
// answers the library's runtime calls.  Device memory is host memory, taken
// from a budget that a test can set; kernels are only recorded.
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

namespace {
std::string g_log;
std::map<const void*, std::string> g_names;
std::map<void*, size_t> g_mem;
size_t g_used = 0, g_budget = size_t(1) << 40;
int g_config[8];
hipStream_t g_stream;
void note(const std::string& s) { g_log += s + "\n"; }
}  // namespace

extern "C" {
const char* host_hip_log() { return g_log.c_str(); }
void host_hip_clear() { g_log.clear(); }
void host_hip_budget(size_t bytes) { g_budget = bytes; }
size_t host_hip_used() { return g_used; }

void** __hipRegisterFatBinary(const void*) {
  static void* handle;
  return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  g_names[f] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t, hipStream_t s) {
  const int c[] = {int(g.x), int(g.y), int(g.z), int(b.x), int(b.y), int(b.z)};
  std::memcpy(g_config, c, sizeof c);
  g_stream = s;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* shmem, hipStream_t* s) {
  *g = dim3(g_config[0], g_config[1], g_config[2]);
  *b = dim3(g_config[3], g_config[4], g_config[5]);
  *shmem = 0;
  *s = g_stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t, hipStream_t) {
  char buf[256];
  std::snprintf(buf, sizeof buf, " grid %u %u %u block %u", g.x, g.y, g.z, b.x);
  std::string s = "launch " + g_names[f] + buf;
  if (s.find("fused_kernel") != std::string::npos) {  // KernelArgs: M, S, n, run
    const int* a = static_cast<const int*>(args[0]);
    std::snprintf(buf, sizeof buf, " n %d run %d", a[2], a[3]);
    s += buf;
  }
  note(s);
  return hipSuccess;
}

hipError_t hipMalloc(void** p, size_t n) {
  if (n > g_budget || g_used > g_budget - n) {
    note("malloc refused");
    return hipErrorOutOfMemory;
  }
  *p = std::malloc(n ? n : 1);
  g_mem[*p] = n;
  g_used += n;
  note("malloc");
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  g_used -= g_mem[p];
  g_mem.erase(p);
  std::free(p);
  note("free");
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  std::memcpy(d, s, n);
  note("memcpy");
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  std::memcpy(d, s, n);
  note("memcpy async");
  return hipSuccess;
}
hipError_t hipMemset(void* p, int v, size_t n) {
  std::memset(p, v, n);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) {
  note("synchronize");
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
  *v = 256;
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipMemGetAddressRange(hipDeviceptr_t*, size_t*, hipDeviceptr_t) { return hipErrorNotFound; }
#undef hipPointerGetAttributes
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void*) {
  std::memset(a, 0, sizeof *a);
  a->type = hipMemoryTypeDevice;
  return hipSuccess;
}
}
