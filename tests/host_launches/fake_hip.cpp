// A stand-in for the HIP runtime that runs nothing: device memory is host
// memory, kernel launches are written down with their grid and first
// arguments, occupancy is what the check says, and an allocation fails when
// the check asks for it.  The library's host layer can be driven with it
// where there is no GPU.
#include <cxxabi.h>

#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {

struct Launch {
  std::string kernel;
  uint32_t grid[3], block[3];
  uint64_t args[16];
};
std::map<const void*, std::string> g_names;
std::vector<Launch> g_launches;
std::vector<std::string> g_queries;                    // kernels of occupancy queries
std::vector<std::pair<std::string, int>> g_occupancy;  // substring, blocks
std::map<std::string, int> g_n_args;
long long g_fail_malloc = -1;                          // mallocs until one fails
int g_set_attribute = 0;
int g_frees = 0;                                       // of device memory
int g_last_error = 0;

std::string name_of(const void* f) {
  const auto it = g_names.find(f);
  return it == g_names.end() ? "?" : it->second;
}

struct Dim {
  uint32_t x, y, z;
};

int launch(const void* f, Dim grid, Dim block, void** args) {
  // (work items per dimension are 32-bit, and a launch past that is refused)
  if ((uint64_t)grid.x * block.x >= (1ull << 32) || (uint64_t)grid.y * block.y >= (1ull << 32) ||
      grid.x == 0 || grid.y == 0 || grid.z == 0)
    return g_last_error = 9;   // hipErrorInvalidConfiguration
  Launch l{name_of(f), {grid.x, grid.y, grid.z}, {block.x, block.y, block.z}, {}};
  for (const auto& n : g_n_args)
    if (l.kernel.find(n.first) != std::string::npos)
      for (int i = 0; i < n.second && i < 16; ++i) std::memcpy(&l.args[i], args[i], 8);
  g_launches.push_back(l);
  return 0;
}

}  // namespace

extern "C" {

// ---- what a check reads and sets ----
void fake_clear() {
  g_launches.clear();
  g_queries.clear();
  g_set_attribute = 0;
}
int fake_launches() { return (int)g_launches.size(); }
const char* fake_kernel(int i) { return g_launches[i].kernel.c_str(); }
uint32_t fake_grid(int i, int d) { return g_launches[i].grid[d]; }
uint32_t fake_block(int i, int d) { return g_launches[i].block[d]; }
uint64_t fake_arg(int i, int a) { return g_launches[i].args[a]; }
int fake_queries() { return (int)g_queries.size(); }
const char* fake_query(int i) { return g_queries[i].c_str(); }
void fake_occupancy(const char* part, int blocks) { g_occupancy.push_back({part, blocks}); }
void fake_keep_args(const char* part, int n) { g_n_args[part] = n; }
void fake_fail_malloc(long long after) { g_fail_malloc = after; }
int fake_frees() { return g_frees; }
int fake_set_attribute() { return g_set_attribute; }

// ---- the runtime ----
void** __hipRegisterFatBinary(const void*) {
  static void* h;
  return &h;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* device, unsigned, void*,
                           void*, void*, void*, int*) {
  int st = 0;
  char* d = abi::__cxa_demangle(device, nullptr, nullptr, &st);
  g_names[host] = st == 0 ? d : device;
  std::free(d);
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}

struct Config {
  Dim grid, block;
  size_t shmem;
  void* stream;
};
static std::vector<Config> g_config;
int __hipPushCallConfiguration(Dim grid, Dim block, size_t shmem, void* stream) {
  g_config.push_back({grid, block, shmem, stream});
  return 0;
}
int __hipPopCallConfiguration(Dim* grid, Dim* block, size_t* shmem, void** stream) {
  const Config c = g_config.back();
  g_config.pop_back();
  *grid = c.grid, *block = c.block, *shmem = c.shmem, *stream = c.stream;
  return 0;
}
int hipLaunchKernel(const void* f, Dim grid, Dim block, void** args, size_t, void*) {
  return launch(f, grid, block, args);
}
int hipExtLaunchKernel(const void* f, Dim grid, Dim block, void** args, size_t, void*, void*,
                       void*, int) {
  return launch(f, grid, block, args);
}
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int, size_t) {
  const std::string k = name_of(f);
  g_queries.push_back(k);
  *n = 2;
  for (const auto& o : g_occupancy)
    if (k.find(o.first) != std::string::npos) *n = o.second;
  return 0;
}
int hipFuncSetAttribute(const void*, int, int) {
  ++g_set_attribute;
  return 0;
}
int hipMalloc(void** p, size_t bytes) {
  *p = nullptr;
  if (g_fail_malloc >= 0 && g_fail_malloc-- == 0) return g_last_error = 2;   // out of memory
  *p = std::calloc(1, bytes + 256);
  return *p ? 0 : 2;
}
int hipFree(void* p) {
  ++g_frees;
  std::free(p);
  return 0;
}
int hipMemcpy(void* d, const void* s, size_t n, int) {
  std::memcpy(d, s, n);
  return 0;
}
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void*) {
  std::memcpy(d, s, n);
  return 0;
}
int hipGetSymbolAddress(void** p, const void*) {
  static void* scratch = std::calloc(1, 16 << 20);
  *p = scratch;
  return 0;
}
int hipDeviceGetAttribute(int* v, int, int) {
  *v = 256;
  return 0;
}
int hipGetDevice(int* d) {
  *d = 0;
  return 0;
}
int hipGetLastError() {
  const int e = g_last_error;
  g_last_error = 0;
  return e;
}
const char* hipGetErrorString(int) { return "an error of the stand-in"; }
static int handle(void** h) {
  *h = std::malloc(8);
  return 0;
}
int hipEventCreate(void** e) { return handle(e); }
int hipEventCreateWithFlags(void** e, unsigned) { return handle(e); }
int hipEventDestroy(void* e) {
  std::free(e);
  return 0;
}
int hipEventElapsedTime(float* ms, void*, void*) {
  *ms = 1.f;
  return 0;
}
int hipEventRecord(void*, void*) { return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipStreamCreateWithFlags(void** s, unsigned) { return handle(s); }
int hipStreamDestroy(void* s) {
  std::free(s);
  return 0;
}
int hipStreamSynchronize(void*) { return 0; }
int hipStreamWaitEvent(void*, void*, unsigned) { return 0; }
int hipStreamBeginCapture(void*, int) { return 0; }
int hipStreamEndCapture(void*, void** g) { return handle(g); }
int hipGraphDestroy(void* g) {
  std::free(g);
  return 0;
}
int hipGraphExecDestroy(void* g) {
  std::free(g);
  return 0;
}
int hipGraphInstantiate(void** x, void*, void**, char*, size_t) { return handle(x); }
int hipGraphLaunch(void*, void*) { return 0; }

}  // extern "C"
