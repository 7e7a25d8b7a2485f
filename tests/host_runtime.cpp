// A stand-in for the HIP runtime in host memory, for tests of the library's
// host code on a machine without a GPU: buffers are host memory, a launch is
// recorded and runs nothing, and one chosen call can be made to fail. Loaded
// with global symbols before libpmfem.so, whose calls then resolve to it.
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

namespace {

struct Dim3 {
  uint32_t x, y, z;
};
struct Watch {
  std::string kernel;
  int arg;
  std::vector<uint64_t> seen;
};

constexpr size_t kLdsDefault = 65536;   // dynamic LDS of a kernel without an attribute
constexpr int kLds = 163840;            // LDS of a workgroup
constexpr int kFail = 2;                // hipErrorOutOfMemory

std::mutex mu;
std::map<const void*, std::string> names;
std::map<const void*, size_t> limit;
std::map<std::string, int64_t> launches, attributes;
std::vector<Watch> watches;
std::string over;      // kernels launched over their limit
std::string fail_call;
int64_t fail_in = 0;     // calls of fail_call until the first that fails (0: none)
int64_t fail_more = 0;   // and how many fail from then on
Dim3 cfg_grid, cfg_block;
size_t cfg_lds;
void* cfg_stream;

int call(const char* what) {
  std::lock_guard<std::mutex> lock(mu);
  if (fail_call != what || fail_more == 0 || (fail_in > 0 && --fail_in > 0)) return 0;
  --fail_more;
  return kFail;
}

int get(void** p, size_t n, const char* what) {
  *p = nullptr;
  if (const int e = call(what)) return e;
  *p = std::calloc(n ? n : 1, 1);
  return *p ? 0 : kFail;
}

int64_t count(const std::map<std::string, int64_t>& m, const char* kernel) {
  int64_t n = 0;
  for (const auto& l : m)
    if (l.first.find(kernel) != std::string::npos) n += l.second;
  return n;
}

}  // namespace

extern "C" {

// -- for the tests ---------------------------------------------------------
void stub_fail_run(const char* what, int64_t nth, int64_t calls) {
  fail_call = what;
  fail_in = nth;
  fail_more = calls;
}
void stub_fail(const char* what, int64_t nth) { stub_fail_run(what, nth, 1); }
int stub_failed() { return fail_in == 0; }
const char* stub_over() { return over.c_str(); }
int stub_watch(const char* kernel, int arg) {
  watches.push_back({kernel, arg, {}});
  return (int)watches.size() - 1;
}
int64_t stub_seen(int w, uint64_t* out, int64_t cap) {
  const auto& s = watches[w].seen;
  for (size_t i = 0; i < s.size() && (int64_t)i < cap; ++i) out[i] = s[i];
  return (int64_t)s.size();
}
int64_t stub_launches(const char* kernel) { return count(launches, kernel); }
int64_t stub_attributes(const char* kernel) { return count(attributes, kernel); }

// -- the runtime -----------------------------------------------------------
void** __hipRegisterFatBinary(const void*) {
  static void* handle;
  return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*,
                           void*, void*, int*) {
  names[f] = name;
}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void* stream) {
  cfg_grid = grid;
  cfg_block = block;
  cfg_lds = lds;
  cfg_stream = stream;
  return 0;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* lds, void** stream) {
  *grid = cfg_grid;
  *block = cfg_block;
  *lds = cfg_lds;
  *stream = cfg_stream;
  return 0;
}
int hipLaunchKernel(const void* f, Dim3 grid, Dim3 block, void** args, size_t lds, void*) {
  std::lock_guard<std::mutex> lock(mu);
  const std::string& name = names[f];
  ++launches[name];
  const auto l = limit.find(f);
  if (lds > (l == limit.end() ? kLdsDefault : l->second) || block.x == 0 || grid.x == 0 ||
      (uint64_t)block.x * block.y * block.z > 1024)
    over += name + " " + std::to_string(lds) + "\n";
  for (Watch& w : watches)
    if (name.find(w.kernel) != std::string::npos) {
      uint64_t v;
      std::memcpy(&v, args[w.arg], sizeof v);
      w.seen.push_back(v);
    }
  return 0;
}
int hipFuncSetAttribute(const void* f, int, int value) {
  ++attributes[names[f]];
  limit[f] = (size_t)value;
  return 0;
}
int hipGetDeviceCount(int* n) {
  *n = 1;
  return 0;
}
int hipGetDevice(int* d) {
  *d = 0;
  return 0;
}
int hipSetDevice(int) { return 0; }
int hipDeviceGetAttribute(int* v, int, int) {
  *v = kLds;
  return 0;
}
const char* hipGetErrorString(int) { return "refused by the test"; }
int hipGetLastError() { return 0; }
int hipGetSymbolAddress(void** p, const void*) {
  static uint64_t word;
  *p = &word;
  return 0;
}
int hipMalloc(void** p, size_t n) { return get(p, n, "hipMalloc"); }
int hipFree(void* p) {
  std::free(p);
  return 0;
}
int hipHostMalloc(void** p, size_t n, unsigned) { return get(p, n, "hipHostMalloc"); }
int hipHostFree(void* p) {
  std::free(p);
  return 0;
}
int hipHostGetDevicePointer(void** d, void* h, unsigned) {
  if (const int e = call("hipHostGetDevicePointer")) return e;
  *d = h;
  return 0;
}
int hipMemcpy(void* d, const void* s, size_t n, int) {
  if (const int e = call("hipMemcpy")) return e;
  std::memcpy(d, s, n);
  return 0;
}
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void*) {
  std::memcpy(d, s, n);
  return 0;
}
int hipMemset(void* d, int v, size_t n) {
  std::memset(d, v, n);
  return 0;
}
int hipMemsetAsync(void* d, int v, size_t n, void*) {
  std::memset(d, v, n);
  return 0;
}
int hipStreamCreateWithFlags(void** s, unsigned) { return get(s, 1, "hipStreamCreateWithFlags"); }
int hipStreamDestroy(void* s) {
  std::free(s);
  return 0;
}
int hipStreamSynchronize(void*) { return 0; }
int hipStreamWaitEvent(void*, void*, unsigned) { return 0; }
int hipEventCreate(void** e) { return get(e, 1, "hipEventCreate"); }
int hipEventCreateWithFlags(void** e, unsigned) { return get(e, 1, "hipEventCreateWithFlags"); }
int hipEventDestroy(void* e) {
  std::free(e);
  return 0;
}
int hipEventRecord(void*, void*) { return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*) {
  *ms = 1.f;
  return 0;
}
}
