// A stand-in for the HIP runtime calls of the library, for host tests without a GPU: "device"
// memory is host memory, copies copy at once, kernels do not run - a launch is written down
// as a line "name grid block lds".  Host allocations of pinned memory can be made to fail.
#include <cxxabi.h>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

namespace {
struct Dim {
  uint32_t x, y, z;
};
struct Config {
  Dim grid, block;
  size_t lds;
  void* stream;
};
std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> m;
  return m;
}
Config pushed;
std::string text;
int fail_pinned, pinned_calls, last_error;
double symbol[1 << 16];
int handle;
constexpr int kOutOfMemory = 2;
}  // namespace

extern "C" {
// ---- for the tests ----
const char* stub_launches() { return text.c_str(); }
void stub_clear() { text.clear(); }
void stub_fail_pinned(int on) { fail_pinned = on; }
int stub_pinned_calls() { return pinned_calls; }

// ---- what the compiler's host code calls ----
void** __hipRegisterFatBinary(const void*) {
  static void* module;
  return &module;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  int status = 0;
  char* plain = abi::__cxa_demangle(name, nullptr, nullptr, &status);
  names()[host] = plain ? plain : name;
  free(plain);
}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim grid, Dim block, size_t lds, void* stream) {
  pushed = Config{grid, block, lds, stream};
  return 0;
}
int __hipPopCallConfiguration(Dim* grid, Dim* block, size_t* lds, void** stream) {
  *grid = pushed.grid;
  *block = pushed.block;
  *lds = pushed.lds;
  *stream = pushed.stream;
  return 0;
}
int hipLaunchKernel(const void* host, Dim g, Dim b, void**, size_t lds, void*) {
  char line[64];
  std::snprintf(line, sizeof line, " %ux%ux%u %ux%ux%u %zu\n", g.x, g.y, g.z, b.x, b.y, b.z, lds);
  std::string n = names()[host];
  n = n.substr(0, n.find('('));
  for (std::string cut : {"void ", "choco::"}) {
    const size_t at = n.find(cut);
    if (at != std::string::npos) n.erase(at, cut.size());
  }
  std::string tight;
  for (char c : n)
    if (c != ' ') tight += c;
  text += tight + line;
  return 0;
}

// ---- runtime ----
int hipGetLastError() {
  const int e = last_error;
  last_error = 0;
  return e;
}
int hipHostMalloc(void** p, size_t n, unsigned) {
  ++pinned_calls;
  if (fail_pinned) return last_error = kOutOfMemory;
  *p = std::calloc(1, n);
  return 0;
}
int hipHostFree(void* p) { return std::free(p), 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void*) { return std::memcpy(d, s, n), 0; }
int hipMemcpy2DAsync(void* d, size_t dp, const void* s, size_t sp, size_t w, size_t h, int, void*) {
  for (size_t r = 0; r < h; ++r) std::memcpy((char*)d + r * dp, (const char*)s + r * sp, w);
  return 0;
}
int hipMemsetAsync(void* d, int v, size_t n, void*) { return std::memset(d, v, n), 0; }
int hipGetSymbolAddress(void** p, const void*) { return *p = symbol, 0; }
int hipGetDevice(int* d) { return *d = 0, 0; }
int hipStreamCreateWithFlags(void** s, unsigned) { return *s = &handle, 0; }
int hipStreamDestroy(void*) { return 0; }
int hipStreamSynchronize(void*) { return 0; }
int hipStreamWaitEvent(void*, void*, unsigned) { return 0; }
int hipEventCreate(void** e) { return *e = &handle, 0; }
int hipEventCreateWithFlags(void** e, unsigned) { return *e = &handle, 0; }
int hipEventDestroy(void*) { return 0; }
int hipEventRecord(void*, void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*) { return *ms = 0.0f, 0; }
}
