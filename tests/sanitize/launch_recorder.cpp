// A HIP runtime that launches nothing and keeps the names and grids of the kernels it is asked for, so that the host side of
// the library shows on the CPU which kernels a call takes.  Linked with the library's host objects, whose device code is not
// built.
#include <cxxabi.h>
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <map>
#include <string>

namespace {
std::map<const void *, std::string> &kernels() {
  static std::map<const void *, std::string> k;
  return k;
}
std::string &record() {
  static std::string r;
  return r;
}
struct Configuration { dim3 grid, block; size_t lds; hipStream_t stream; };
Configuration pushed;
}  // namespace

extern "C" {
extern const char __hip_fatbin[8];
const char __hip_fatbin[8] = {0};

void **__hipRegisterFatBinary(const void *) {
  static void *module;
  return &module;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, dim3 *, dim3 *, int *) {
  int status = 0;
  char *plain = abi::__cxa_demangle(name, nullptr, nullptr, &status);
  std::string s = status == 0 ? plain : name;
  std::free(plain);
  if (s.rfind("void ", 0) == 0) s = s.substr(5);
  for (const char *drop : {"rsa::", "(anonymous namespace)::"})
    for (size_t at; (at = s.find(drop)) != std::string::npos;) s.erase(at, std::string(drop).size());
  kernels()[host] = s.substr(0, s.find('('));
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream) {
  pushed = {grid, block, lds, stream};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *stream) {
  *grid = pushed.grid; *block = pushed.block; *lds = pushed.lds; *stream = pushed.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void *kernel, dim3 grid, dim3 block, void **, size_t, hipStream_t) {
  char sizes[96];
  std::snprintf(sizes, sizeof(sizes), "|%u,%u,%u|%u\n", grid.x, grid.y, grid.z, block.x);
  record() += kernels()[kernel] + sizes;
  return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipGetDevice(int *device) { *device = 0; return hipSuccess; }
hipError_t hipGetSymbolAddress(void **address, const void *) { *address = reinterpret_cast<void *>(0x1000000); return hipSuccess; }

// What was launched since the last call of this function: a line `name|grid|threads` each.
__attribute__((visibility("default"))) const char *launches(void) {
  static std::string last;
  last.swap(record());
  record().clear();
  return last.c_str();
}
}
