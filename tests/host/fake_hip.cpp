// A HIP runtime for the library's host code alone: device memory is host memory
// with an optional limit, kernels are not run but listed (name and grid) in the
// order of their launches.  Loaded ahead of libpsdf.so, whose calls then come
// here; tests of plans, routes and refusals use it where there is no GPU.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {
struct Dim3 {
  uint32_t x, y, z;
};
struct Config {
  Dim3 grid, block;
  size_t shmem;
  void* stream;
};
constexpr int kOk = 0, kOutOfMemory = 2;
std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> m;
  return m;
}
std::map<void*, size_t> blocks;
size_t used = 0, limit = ~size_t(0);
long fail_at = -1, mallocs = 0, launched = 0;
int last_error = kOk;
std::vector<Config> configs;
std::string launches;
char handle[64], symbol[8 << 20];

void note(const void* f, Dim3 g, Dim3 b) {
  char buf[96];
  std::snprintf(buf, sizeof buf, " %u %u %u\n", g.x, g.y, b.x);
  launches += names()[f] + buf;
  ++launched;
}
}  // namespace

extern "C" {
// ---- the tests' own calls
void fake_limit(size_t bytes) { limit = bytes; }
void fake_fail_malloc(long k) { fail_at = k < 0 ? -1 : mallocs + k; }   // the k-th from now
size_t fake_used() { return used; }
const char* fake_launches() { return launches.c_str(); }
void fake_clear() { launches.clear(); }

// ---- the runtime
int hipMalloc(void** p, size_t n) {
  *p = nullptr;
  if (mallocs++ == fail_at || used > limit || n > limit - used) return last_error = kOutOfMemory;
  *p = std::calloc(1, n ? n : 1);
  blocks[*p] = n;
  used += n;
  return kOk;
}
int hipFree(void* p) {
  if (!p) return kOk;
  used -= blocks.at(p);
  blocks.erase(p);
  std::free(p);
  return kOk;
}
int hipMemcpy(void* d, const void* s, size_t n, int) {
  std::memcpy(d, s, n);
  return kOk;
}
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void*) { return hipMemcpy(d, s, n, 0); }
int hipMemset(void* d, int v, size_t n) {
  std::memset(d, v, n);
  return kOk;
}
int hipGetLastError() {
  const int e = last_error;
  last_error = kOk;
  return e;
}
int hipGetDevice(int* d) {
  *d = 0;
  return kOk;
}
int hipSetDevice(int) { return kOk; }
int hipDeviceGetAttribute(int* v, int, int) {
  *v = 256;
  return kOk;
}
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
  *n = 8;
  return kOk;
}
int hipGetSymbolAddress(void** p, const void*) {
  *p = symbol;
  return kOk;
}
// a kernel takes a millisecond
int hipEventCreate(void** e) {
  *e = new long(0);
  return kOk;
}
int hipEventCreateWithFlags(void** e, unsigned) { return hipEventCreate(e); }
int hipEventDestroy(void* e) {
  delete static_cast<long*>(e);
  return kOk;
}
int hipEventRecord(void* e, void*) {
  *static_cast<long*>(e) = launched;
  return kOk;
}
int hipEventSynchronize(void*) { return kOk; }
int hipEventElapsedTime(float* ms, void* a, void* b) {
  *ms = (float)(*static_cast<long*>(b) - *static_cast<long*>(a));
  return kOk;
}
int hipStreamCreateWithFlags(void** s, unsigned) {
  *s = handle;
  return kOk;
}
int hipStreamDestroy(void*) { return kOk; }
int hipStreamWaitEvent(void*, void*, unsigned) { return kOk; }
int hipStreamBeginCapture(void*, int) { return kOk; }
int hipStreamEndCapture(void*, void** g) {
  *g = handle;
  return kOk;
}
int hipGraphInstantiate(void** e, void*, void*, char*, size_t) {
  *e = handle;
  return kOk;
}
int hipGraphLaunch(void*, void*) { return kOk; }
int hipGraphDestroy(void*) { return kOk; }
int hipGraphExecDestroy(void*) { return kOk; }

int hipLaunchKernel(const void* f, Dim3 grid, Dim3 block, void**, size_t, void*) {
  note(f, grid, block);
  return kOk;
}
int hipExtLaunchKernel(const void* f, Dim3 grid, Dim3 block, void**, size_t, void*, void*, void*,
                       int) {
  note(f, grid, block);
  return kOk;
}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t shmem, void* stream) {
  configs.push_back({grid, block, shmem, stream});
  return kOk;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* shmem, void** stream) {
  const Config c = configs.back();
  configs.pop_back();
  *grid = c.grid;
  *block = c.block;
  *shmem = c.shmem;
  *stream = c.stream;
  return kOk;
}
void** __hipRegisterFatBinary(const void*) {
  static void* module = handle;
  return &module;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*,
                           Dim3*, Dim3*, int*) {
  names()[f] = name;
}
}  // extern "C"
