// A stand-in for the HIP runtime, for tests of the library's host side without a GPU: it registers kernels under their
// names, records every launch instead of running it, checks the dynamic LDS size against what hipFuncSetAttribute allowed,
// and fails a launch or an attribute call on request.  Built as libamdhip64.so.7 and loaded before the library.
#include <chrono>
#include <condition_variable>
#include <cstddef>
#include <cstdint>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

namespace {
struct Dim3 { uint32_t x, y, z; };
struct Launch { std::string name; Dim3 grid, block; size_t lds; };
struct Config { Dim3 grid, block; size_t lds; void* stream; };
std::mutex mu;
std::condition_variable attribute_set;
std::map<const void*, std::string> names;
std::map<const void*, size_t> allowed;
std::vector<Launch> launches;
int fail_launch_in = -1, fail_attribute_in = -1;
bool hold_first = false;
int attribute_calls = 0, attributes_done = 0;
thread_local std::vector<Config> configs;
thread_local int last_error = 0;
constexpr int INVALID_VALUE = 1, OUT_OF_MEMORY = 2;
}  // namespace

extern "C" {
// ---- what the library imports
void** __hipRegisterFatBinary(const void*) { static void* handle; return &handle; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* device, unsigned, void*, void*, void*, void*, int*) {
  std::lock_guard<std::mutex> l(mu);
  names[host] = device;
}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void* stream) {
  configs.push_back({grid, block, lds, stream});
  return 0;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* lds, void** stream) {
  const Config c = configs.back();
  configs.pop_back();
  *grid = c.grid;
  *block = c.block;
  *lds = c.lds;
  *stream = c.stream;
  return 0;
}
int hipLaunchKernel(const void* f, Dim3 grid, Dim3 block, void**, size_t lds, void*) {
  std::lock_guard<std::mutex> l(mu);
  size_t limit = 64 * 1024;
  if (allowed.count(f) && allowed[f] > limit) limit = allowed[f];
  if (lds > limit) return last_error = INVALID_VALUE;
  if (fail_launch_in >= 0 && fail_launch_in-- == 0) return last_error = OUT_OF_MEMORY;
  launches.push_back({names[f], grid, block, lds});
  return 0;
}
// Sets the size when it returns.  With fake_hold_first_attribute, the first call waits for another one to be done first
// (half a second at most: callers that take turns must get through).
int hipFuncSetAttribute(const void* f, int, int value) {
  std::unique_lock<std::mutex> l(mu);
  if (fail_attribute_in >= 0 && fail_attribute_in-- == 0) return last_error = OUT_OF_MEMORY;
  if (++attribute_calls == 1 && hold_first)
    attribute_set.wait_for(l, std::chrono::milliseconds(500), [] { return attributes_done > 0; });
  allowed[f] = (size_t)value;
  ++attributes_done;
  attribute_set.notify_all();
  return 0;
}
int hipGetLastError() { const int e = last_error; last_error = 0; return e; }
const char* hipGetErrorString(int) { return "error of the stand-in runtime"; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int* v, int, int) { *v = 256; return 0; }
int hipGetSymbolAddress(void** p, const void*) { *p = (void*)(uintptr_t)(1ull << 40); return 0; }

// ---- what the tests call
void fake_reset() {
  std::lock_guard<std::mutex> l(mu);
  launches.clear();
  allowed.clear();
  fail_launch_in = fail_attribute_in = -1;
}
void fake_fail_launch(int after) { std::lock_guard<std::mutex> l(mu); fail_launch_in = after; }
void fake_fail_attribute(int after) { std::lock_guard<std::mutex> l(mu); fail_attribute_in = after; }
void fake_hold_first_attribute() {
  std::lock_guard<std::mutex> l(mu);
  hold_first = true;
  attribute_calls = attributes_done = 0;
}
int fake_attribute_calls() { std::lock_guard<std::mutex> l(mu); return attribute_calls; }
int fake_launches() { std::lock_guard<std::mutex> l(mu); return (int)launches.size(); }
const char* fake_name(int i) { std::lock_guard<std::mutex> l(mu); return launches[(size_t)i].name.c_str(); }
uint64_t fake_lds(int i) { std::lock_guard<std::mutex> l(mu); return launches[(size_t)i].lds; }
uint32_t fake_grid(int i, int axis) {
  std::lock_guard<std::mutex> l(mu);
  const Dim3 g = launches[(size_t)i].grid;
  return axis == 0 ? g.x : axis == 1 ? g.y : g.z;
}
}
