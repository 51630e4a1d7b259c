// Stand-in for the HIP runtime calls of the library, to run its host code without a GPU (preloaded by
// test_plan_memory_cpu.py): device memory is host memory, kernels do nothing, allocations and launches go to the file
// HIP_STUB_LOG.  HIP_STUB_FAIL: so many of the next allocations above HIP_STUB_LARGE bytes find no room.
#define __HIP_PLATFORM_AMD__
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

static std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> m;
  return m;
}
static void log_line(const char* what, const std::string& v) {
  static FILE* f = std::getenv("HIP_STUB_LOG") ? std::fopen(std::getenv("HIP_STUB_LOG"), "a") : nullptr;
  if (f) std::fprintf(f, "%s %s\n", what, v.c_str()), std::fflush(f);
}
static long env(const char* n) { return std::getenv(n) ? std::atol(std::getenv(n)) : 0; }

extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
  static long fail = env("HIP_STUB_FAIL");
  const bool large = n > size_t(env("HIP_STUB_LARGE"));
  const bool ok = !(large && fail > 0 && fail--);
  if (large) log_line(ok ? "large" : "refused", std::to_string(n));
  *p = ok ? std::malloc(n) : nullptr;
  return ok ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void* p) { return std::free(p), hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { return std::memcpy(d, s, n), hipSuccess; }
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void* s) { return *p = const_cast<void*>(s), hipSuccess; }
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void**, size_t, hipStream_t) {
  return log_line("launch", names()[f]), hipSuccess;
}
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3*, dim3*, size_t* l, hipStream_t* s) { return *l = 0, *s = nullptr, hipSuccess; }
void** __hipRegisterFatBinary(const void*) {
  static void* handle;
  return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* h, char*, const char* n, unsigned, void*, void*, dim3*, dim3*, int*) {
  names()[h] = n;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
}
