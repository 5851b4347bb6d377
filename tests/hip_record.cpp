// A HIP runtime that records instead of running: what the library asks of the device, seen on a host without one.
// Loaded before the library with RTLD_GLOBAL, its definitions come first.  Addresses are made up by the test:
// bits 40..43 are the device they belong to, bit 44 marks memory the runtime does not know; a stream handle is the
// number of its device.
#include <stddef.h>
#include <stdint.h>

#include <map>
#include <string>

namespace {
std::map<const void*, std::string> g_kernels;
std::string g_calls;
struct Dim3 { uint32_t x, y, z; };
struct Config { Dim3 grid, block; size_t lds; void* stream; } g_config;
struct PointerAttributes {
  int type, device;
  void *device_pointer, *host_pointer;
  int is_managed;
  unsigned flags;
};
int g_last_error = 0;
int g_cus = 256;
int g_launches_until_failure = -1;
}  // namespace

extern "C" {
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  g_kernels[host] = name;
}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void* stream) {
  g_config = Config{grid, block, lds, stream};
  return 0;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* lds, void** stream) {
  *grid = g_config.grid, *block = g_config.block, *lds = g_config.lds, *stream = g_config.stream;
  return 0;
}
int hipLaunchKernel(const void* fn, Dim3 grid, Dim3 block, void**, size_t, void*) {
  if (g_launches_until_failure >= 0 && g_launches_until_failure-- == 0) return g_last_error = 1;
  g_calls += "launch " + g_kernels[fn] + " " + std::to_string((uint64_t)grid.x * grid.y * grid.z) + " " +
             std::to_string((uint64_t)grid.x * block.x) + "\n";
  return 0;
}
int hipMemcpyAsync(void* dst, const void* src, size_t n, int, void*) {
  g_calls += "copy " + std::to_string((uintptr_t)dst) + " " + std::to_string((uintptr_t)src) + " " + std::to_string(n) + "\n";
  return 0;
}
int hipPointerGetAttributes(PointerAttributes* a, const void* p) {
  if ((uintptr_t)p >> 44 & 1) return g_last_error = 1;
  *a = PointerAttributes{2, (int)((uintptr_t)p >> 40 & 15), (void*)p, nullptr, 0, 0};
  return 0;
}
int hipStreamGetDevice(void* stream, int* device) { return *device = (int)(uintptr_t)stream, 0; }
int hipGetDevice(int* device) { return *device = 0, 0; }
int hipDeviceGetAttribute(int* value, int, int) { return *value = g_cus, 0; }
int hipFuncSetAttribute(const void*, int, int) { return 0; }
int hipGetLastError() {
  const int e = g_last_error;
  return g_last_error = 0, e;
}
void record_fail_launch(int after) { g_launches_until_failure = after; }  // the launch after that many more fails
const char* record_take() {
  static std::string taken;
  taken.swap(g_calls);
  g_calls.clear();
  return taken.c_str();
}
}
