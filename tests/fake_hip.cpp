// A stand-in for the HIP runtime's host calls, for tests of the library's
// host code on machines without a GPU: device memory is host memory, kernels
// are recorded and not run. Built with the runtime's soname and loaded before
// libspdp.so, whose calls it then answers.
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <new>
#include <string>

namespace {

constexpr int kInvalid = 1, kOutOfMemory = 2;

struct Dim3 {
  uint32_t x, y, z;
};

// never destroyed: handles may be freed while the process ends
auto& g_names = *new std::map<const void*, std::string>;
auto& g_live = *new std::map<void*, size_t>;
size_t g_budget = ~size_t(0), g_used = 0, g_fail_new = 0;
int g_capturing = 0, g_cus = 256, g_fail_attribute = 0;
auto& g_log = *new std::string;  // one line a call: "malloc BYTES", "malloc-failed BYTES", "launch NAME X Y Z LDS"
Dim3 g_grid, g_block;
size_t g_shared;
void* g_stream;
alignas(256) char g_symbol[(size_t(40) << 20) + 256];

void note(const std::string& line) { g_log += line + "\n"; }

}  // namespace

extern "C" {

// the test's side
void fake_budget(size_t bytes) { g_budget = bytes; }
void fake_capturing(int on) { g_capturing = on; }
void fake_cus(int n) { g_cus = n; }
void fake_fail_attribute(int on) { g_fail_attribute = on; }
void fake_fail_new(size_t bytes) { g_fail_new = bytes; }
size_t fake_used() { return g_used; }
size_t fake_live() { return g_live.size(); }
const char* fake_log() { return g_log.c_str(); }
void fake_clear() { g_log.clear(); }

// the runtime's side
int hipMalloc(void** p, size_t bytes) {
  if (g_used + bytes > g_budget) {
    note("malloc-failed " + std::to_string(bytes));
    return kOutOfMemory;
  }
  *p = std::aligned_alloc(256, (bytes + 255) / 256 * 256);
  if (!*p) return kOutOfMemory;
  g_live[*p] = bytes;
  g_used += bytes;
  note("malloc " + std::to_string(bytes));
  return 0;
}
int hipFree(void* p) {
  const auto it = g_live.find(p);
  if (it == g_live.end()) return kInvalid;
  g_used -= it->second;
  g_live.erase(it);
  std::free(p);
  return 0;
}
int hipMemcpy(void* to, const void* from, size_t bytes, int) {
  std::memcpy(to, from, bytes);
  return 0;
}
int hipMemset(void* p, int v, size_t bytes) {
  std::memset(p, v, bytes);
  return 0;
}
int hipMemsetAsync(void* p, int v, size_t bytes, void*) { return hipMemset(p, v, bytes); }
int hipGetDevice(int* d) {
  *d = 0;
  return 0;
}
int hipSetDevice(int) { return 0; }
int hipDeviceSynchronize() { return 0; }
int hipDeviceGetAttribute(int* v, int, int) {
  *v = g_cus;
  return 0;
}
int hipStreamIsCapturing(void*, int* status) {
  *status = g_capturing;
  return 0;
}
int hipFuncSetAttribute(const void*, int, int) { return g_fail_attribute ? kInvalid : 0; }
int hipGetLastError() { return 0; }
const char* hipGetErrorString(int) { return "an error of the stand-in"; }
int hipGetSymbolAddress(void** p, const void*) {
  *p = g_symbol;
  return 0;
}
int hipLaunchKernel(const void* f, Dim3 grid, Dim3, void**, size_t shared, void*) {
  note("launch " + g_names[f] + " " + std::to_string(grid.x) + " " + std::to_string(grid.y) + " " +
       std::to_string(grid.z) + " " + std::to_string(shared));
  return 0;
}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t shared, void* stream) {
  g_grid = grid;
  g_block = block;
  g_shared = shared;
  g_stream = stream;
  return 0;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* shared, void** stream) {
  *grid = g_grid;
  *block = g_block;
  *shared = g_shared;
  *stream = g_stream;
  return 0;
}
void** __hipRegisterFatBinary(const void*) {
  static void* handle;
  return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*,
                           int*) {
  g_names[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}

}  // extern "C"

// the library's host allocations, of which those of one size can be made to
// fail
void* operator new(size_t bytes) {
  void* p = g_fail_new != 0 && bytes == g_fail_new ? nullptr : std::malloc(bytes ? bytes : 1);
  if (!p) throw std::bad_alloc();
  return p;
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }
