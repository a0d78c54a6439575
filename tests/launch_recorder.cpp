// The HIP calls that libuniql makes, written down instead of carried out: which kernels a call launches, with which grid and LDS, can be
// tested without a GPU.  tests/launches.py builds it and loads it ahead of the library.
#include <hip/hip_runtime_api.h>
#include <map>
#include <string>
#include <stdlib.h>
#include <string.h>
#include <vector>

namespace {
struct Launch {
  std::string kernel;
  long blocks, threads, lds, limit;   // limit: the dynamic LDS that the kernel was allowed when it was launched (0: never set)
};
std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> m;
  return m;
}
std::map<const void*, int> limits;
std::vector<Launch> launches;
dim3 grid, block;
size_t lds;
}  // namespace

extern "C" {
void** __hipRegisterFatBinary(const void*) {
  static void* handle;
  return &handle;
}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { names()[f] = name; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void**) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, hipStream_t) {
  grid = g, block = b, lds = s;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* s, hipStream_t* stream) {
  *g = grid, *b = block, *s = lds, *stream = nullptr;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void**, size_t s, hipStream_t) {
  launches.push_back({names()[f], (long)g.x * g.y * g.z, (long)b.x * b.y * b.z, (long)s, limits.count(f) ? limits[f] : 0});
  return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void* f, hipFuncAttribute, int value) {
  limits[f] = value;
  return hipSuccess;
}
hipError_t hipGetDevice(int* device) {
  *device = 0;
  return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  memset(p, 0, sizeof(*p));
  strcpy(p->gcnArchName, "gfx950");
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* value, hipDeviceAttribute_t, int) {
  const char* cus = getenv("RECORDER_COMPUTE_UNITS");
  *value = cus ? atoi(cus) : 256;
  return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) {
  static char symbol[4096];
  *p = symbol;
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }

int recorded(void) { return (int)launches.size(); }
const char* recorded_kernel(int i) { return launches[i].kernel.c_str(); }
void recorded_sizes(int i, long out[4]) { out[0] = launches[i].blocks, out[1] = launches[i].threads, out[2] = launches[i].lds, out[3] = launches[i].limit; }
void recorded_clear(void) { launches.clear(); }
}
