// Stands in for the HIP runtime under libcure.so, for tests of its launches on the CPU: kernels are
// not run, their names and launch shapes are recorded. A GPU of 256 compute units.
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <map>
#include <string>

namespace {
struct Dim3 {
  uint32_t x, y, z;
};
std::map<const void*, std::string> g_names;
std::string g_log;
int g_capturing = 0;
struct {
  Dim3 grid, block;
  size_t shared;
  void* stream;
} g_config;
}  // namespace

extern "C" {
const char* stub_launches() { return g_log.c_str(); }
void stub_reset(int capturing) {
  g_log.clear();
  g_capturing = capturing;
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
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t shared, void* stream) {
  g_config = {grid, block, shared, stream};
  return 0;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* shared, void** stream) {
  *grid = g_config.grid;
  *block = g_config.block;
  *shared = g_config.shared;
  *stream = g_config.stream;
  return 0;
}
int hipLaunchKernel(const void* host, Dim3 grid, Dim3 block, void**, size_t, void*) {
  char line[128];
  std::snprintf(line, sizeof line, " %u %u %u %u\n", grid.x, grid.y, grid.z, block.x * block.y * block.z);
  g_log += g_names[host] + line;
  return 0;
}
int hipGetLastError() { return 0; }
int hipGetDevice(int* device) { return *device = 0; }
int hipDeviceGetAttribute(int* value, int, int) {
  *value = 256;
  return 0;
}
int hipGetSymbolAddress(void** address, const void*) {
  *address = nullptr;
  return 1;
}
int hipStreamIsCapturing(void*, int* status) {
  *status = g_capturing;
  return 0;
}
}
