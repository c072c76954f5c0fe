// Stands in for the HIP runtime calls of the library (host only): kernels are not run, their
// launches and attribute settings are written down.  Loaded with RTLD_GLOBAL before the
// library, whose calls then resolve here.
#include <stdint.h>
#include <stdio.h>

#include <map>
#include <string>

struct Dim3 { uint32_t x, y, z; };

namespace {
std::string g_log;
std::map<const void*, std::string> g_names;
struct { Dim3 grid, block; size_t lds; void* stream; } g_call;
char g_module, g_array;
}  // namespace

extern "C" {

const char* recorder_log() { return g_log.c_str(); }
void recorder_clear() { g_log.clear(); }

void** __hipRegisterFatBinary(const void*) { static void* m = &g_module; return &m; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, Dim3*, Dim3*, int*) {
  g_names[host] = name;
}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void* stream) {
  g_call = {grid, block, lds, stream};
  return 0;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* lds, void** stream) {
  *grid = g_call.grid; *block = g_call.block; *lds = g_call.lds; *stream = g_call.stream;
  return 0;
}
int hipLaunchKernel(const void* f, Dim3 grid, Dim3 block, void**, size_t lds, void*) {
  char line[160];
  snprintf(line, sizeof line, " %u %u %u %u %zu\n", grid.x, grid.y, grid.z, block.x, lds);
  g_log += "launch " + g_names[f] + line;
  return 0;
}
int hipFuncSetAttribute(const void* f, int attribute, int value) {
  char line[64];
  snprintf(line, sizeof line, " %d %d\n", attribute, value);
  g_log += "attribute " + g_names[f] + line;
  return 0;
}
int hipGetLastError() { return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetSymbolAddress(void** p, const void*) { *p = &g_array; return 0; }
int hipEventCreate(void**) { return 1; }
int hipEventRecord(void*, void*) { return 1; }
int hipEventSynchronize(void*) { return 1; }
int hipEventElapsedTime(float*, void*, void*) { return 1; }

}  // extern "C"
