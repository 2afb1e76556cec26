// A HIP runtime without a GPU, for tests of what the library's host code asks of it: the kernels
// it launches (name, grid, block, first words of the arguments) and the memory it allocates.
// Nothing is executed.  Loaded with RTLD_GLOBAL before libpolymul.so, whose HIP calls then come
// here; "device" memory is host memory, and launches that a dispatch packet cannot hold (a grid
// of 2^32 work-items or more along a dimension) are refused as the real runtime refuses them.
#include <stdint.h>
#include <stdio.h>
#include <string.h>
#include <sys/mman.h>

#include <map>
#include <string>
#include <vector>

namespace {
struct Dim3 { uint32_t x, y, z; };
std::map<const void*, std::string> g_names;
std::map<void*, uint64_t> g_blocks;
uint64_t g_limit = ~0ull, g_used = 0, g_peak = 0;
int g_error = 0;
std::string g_log;
struct Config { Dim3 grid, block; uint64_t lds; void* stream; };
std::vector<Config> g_configs;
int fail(int e) { return g_error = e; }
}  // namespace

extern "C" {

// ---- control, for the test
void fake_hip_reset(uint64_t limit) { g_log.clear(); g_limit = limit; g_peak = g_used; g_error = 0; }
const char* fake_hip_log() { return g_log.c_str(); }  // one launch a line
uint64_t fake_hip_peak() { return g_peak; }
uint64_t fake_hip_used() { return g_used; }

// ---- the runtime
void** __hipRegisterFatBinary(const void*) { static void* handle; return &handle; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  g_names[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void* stream) {
  g_configs.push_back({grid, block, lds, stream});
  return 0;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* lds, void** stream) {
  const Config c = g_configs.back();
  g_configs.pop_back();
  *grid = c.grid; *block = c.block; *lds = c.lds; *stream = c.stream;
  return 0;
}
int hipLaunchKernel(const void* fn, Dim3 grid, Dim3 block, void** args, size_t lds, void*) {
  const auto it = g_names.find(fn);
  if (it == g_names.end()) return fail(98);  // hipErrorInvalidDeviceFunction
  const uint32_t g[3] = {grid.x, grid.y, grid.z}, b[3] = {block.x, block.y, block.z};
  for (int d = 0; d < 3; ++d)
    if (!g[d] || !b[d] || (uint64_t)g[d] * b[d] >> 32) return fail(9);  // hipErrorInvalidConfiguration
  if ((uint64_t)b[0] * b[1] * b[2] > 1024 || lds > 160 * 1024) return fail(9);
  char buf[160];
  snprintf(buf, sizeof buf, " %u %u %u %zu", g[0], g[1], b[0], lds);
  g_log += it->second + buf;
  if (it->second.find("ptrans") != std::string::npos || it->second.find("pt_outer") != std::string::npos) {
    uint64_t w[8];  // these kernels take one structure larger than this, pointers first
    memcpy(w, args[0], sizeof w);
    for (uint64_t v : w) {
      snprintf(buf, sizeof buf, " %llu", (unsigned long long)v);
      g_log += buf;
    }
  }
  g_log += "\n";
  return 0;
}
int hipGetLastError() { const int e = g_error; g_error = 0; return e; }
const char* hipGetErrorString(int) { return "fake"; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetDevicePropertiesR0600(void*, int) { return 1; }  // the library then takes 256 CUs
int hipFuncSetAttribute(const void*, int, int) { return 0; }
int hipGetSymbolAddress(void** p, const void*) { *p = (void*)0x700000000000ull; return 0; }
int hipMalloc(void** p, size_t bytes) {
  if (bytes > g_limit || g_used > g_limit - bytes) return fail(2);  // hipErrorOutOfMemory
  void* m = mmap(nullptr, bytes ? bytes : 1, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  if (m == MAP_FAILED) return fail(2);
  g_blocks[m] = bytes;
  g_used += bytes;
  if (g_used > g_peak) g_peak = g_used;
  *p = m;
  return 0;
}
int hipFree(void* p) {
  const auto it = g_blocks.find(p);
  if (it == g_blocks.end()) return fail(1);
  g_used -= it->second;
  munmap(p, it->second ? it->second : 1);
  g_blocks.erase(it);
  return 0;
}
int hipMemcpy(void* d, const void* s, size_t n, int) { memcpy(d, s, n); return 0; }
int hipMemset(void* d, int v, size_t n) { memset(d, v, n); return 0; }
int hipStreamSynchronize(void*) { return 0; }
int hipStreamCreateWithFlags(void** s, unsigned) { *s = (void*)1; return 0; }
int hipStreamDestroy(void*) { return 0; }
int hipStreamBeginCapture(void*, int) { return 0; }
int hipStreamEndCapture(void*, void** g) { *g = (void*)1; return 0; }
int hipGraphInstantiate(void** e, void*, void*, char*, size_t) { *e = (void*)1; return 0; }
int hipGraphLaunch(void*, void*) { return 0; }
int hipGraphDestroy(void*) { return 0; }
int hipGraphExecDestroy(void*) { return 0; }

}  // extern "C"
