// The few HIP calls that libmg5mi.so makes, without a GPU: launches are
// recorded instead of made.  test_launches_host.py loads this library ahead of
// the HIP runtime, so that the host code that cuts and dispatches launches runs
// on the CPU at sizes that no test could allocate.
#include <cstddef>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

struct dim3 {
  uint32_t x, y, z;
};
struct Launch {
  const char* kernel;
  uint32_t grid, block;
  uint64_t args[3];  // the first three arguments, eight bytes each
};
static std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> m;
  return m;
}
static std::vector<Launch>& launches() {
  static std::vector<Launch> v;
  return v;
}
static dim3 grid, block;

extern "C" {
void** __hipRegisterFatBinary(const void*) { return (void**)std::calloc(1, 8); }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*,
                           void*, void*, int*) {
  names()[f] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t, void*) {
  grid = g;
  block = b;
  return 0;
}
int __hipPopCallConfiguration(dim3* g, dim3* b, size_t* shared, void** stream) {
  *g = grid;
  *b = block;
  *shared = 0;
  *stream = nullptr;
  return 0;
}
int hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t, void*) {
  Launch l{names()[f].c_str(), g.x, b.x, {}};
  for (int k = 0; k < 3; ++k) std::memcpy(&l.args[k], args[k], 8);  // every kernel has three
  launches().push_back(l);
  return 0;
}
int hipMalloc(void** p, size_t n) {
  *p = std::malloc(n);
  return *p ? 0 : 2;
}
int hipFree(void* p) {
  std::free(p);
  return 0;
}
// what the helicity filter reads back: every helicity contributes
int hipMemcpy(void* to, const void*, size_t n, int) {
  for (size_t k = 0; k < n / sizeof(double); ++k) ((double*)to)[k] = 1.0;
  return 0;
}
int hipGetLastError() { return 0; }
int hipGetDevice(int* d) {
  *d = 0;
  return 0;
}
int hipGetSymbolAddress(void** p, const void*) {
  *p = (void*)4096;
  return 0;
}

int record_count() { return (int)launches().size(); }
void record_clear() { launches().clear(); }
const char* record_kernel(int k) { return launches()[k].kernel; }
uint32_t record_grid(int k) { return launches()[k].grid; }
uint32_t record_block(int k) { return launches()[k].block; }
uint64_t record_arg(int k, int a) { return launches()[k].args[a]; }
}
