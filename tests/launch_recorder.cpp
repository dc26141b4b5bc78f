// Stands in for the HIP runtime in a process without a GPU: device memory is never touched, copies do
// nothing, and every kernel launch is recorded with its name, grid, workgroup and dynamic LDS, and with the LDS
// limit that hipFuncSetAttribute had raised for that kernel before.
#include <cstdint>
#include <cstdlib>
#include <map>
#include <string>
#include <vector>

struct Dim3 { uint32_t x, y, z; };
struct Launch { const char* name; Dim3 grid, block; size_t lds, limit; };
static std::map<const void*, std::string>& names() { static std::map<const void*, std::string> m; return m; }
static std::map<const void*, size_t> limits;
static std::vector<Launch> launches;
static struct { Dim3 grid, block; size_t lds; void* stream; } pushed;

extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* handle; return &handle; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* stub, char* name, const char*, unsigned, void*, void*, void*, void*, int*) {
  names()[stub] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void* stream) { pushed = {grid, block, lds, stream}; return 0; }
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* lds, void** stream) {
  *grid = pushed.grid; *block = pushed.block; *lds = pushed.lds; *stream = pushed.stream;
  return 0;
}
int hipLaunchKernel(const void* stub, Dim3 grid, Dim3 block, void**, size_t lds, void*) {
  const auto l = limits.find(stub);
  launches.push_back({names()[stub].c_str(), grid, block, lds, l == limits.end() ? 0 : l->second});
  return 0;
}
int hipFuncSetAttribute(const void* stub, int attribute, int value) {
  if (attribute == 8) limits[stub] = (size_t)value;      // the largest dynamic LDS size
  return 0;
}
int hipDeviceGetAttribute(int* value, int, int) { *value = 256; return 0; }
int hipGetDevice(int* device) { *device = 0; return 0; }
int hipGetLastError() { return 0; }
const char* hipGetErrorString(int) { return "recorded"; }
int hipGetSymbolAddress(void** at, const void*) { *at = (void*)((uintptr_t)1 << 32); return 0; }
int hipHostMalloc(void** at, size_t n, unsigned) { *at = calloc(1, n); return *at ? 0 : 2; }
int hipHostFree(void* at) { free(at); return 0; }
int hipMemcpyAsync(void*, const void*, size_t, int, void*) { return 0; }
int hipStreamSynchronize(void*) { return 0; }
int hipEventCreate(void** e) { *e = nullptr; return 0; }
int hipEventDestroy(void*) { return 0; }
int hipEventRecord(void*, void*) { return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*) { *ms = 0.f; return 0; }

void recorded_clear() { launches.clear(); }
int recorded_count() { return (int)launches.size(); }
const char* recorded_at(int i, uint64_t* out) {
  const Launch& l = launches[i];
  const uint64_t v[8] = {l.grid.x, l.grid.y, l.grid.z, l.block.x, l.block.y, l.block.z, l.lds, l.limit};
  for (int j = 0; j < 8; ++j) out[j] = v[j];
  return l.name;
}
}
