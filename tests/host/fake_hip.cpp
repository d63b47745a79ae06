// A stand-in for the HIP runtime calls of libsk.so, so that what the library
// allocates and launches can be tested without a GPU. Loaded with RTLD_GLOBAL before
// libsk.so, whose calls then come here. Device memory is addresses only, nothing runs;
// every call that matters is a line of the log.
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include <atomic>
#include <map>
#include <mutex>
#include <string>

namespace {
std::mutex mu;
std::map<const void*, std::string> kernels;
std::map<uintptr_t, size_t> blocks;
std::string text;
size_t used = 0, limit = (size_t)1 << 48;
uintptr_t next_block = 0x7f0000000000ull;
std::atomic<int> events_done{1}, cus{256};
uint8_t symbols[64];
size_t n_symbols = 0;
struct Dim {
  uint32_t x, y, z;
};
thread_local Dim cfg_grid, cfg_block;
thread_local size_t cfg_lds;
thread_local void* cfg_stream;

void log(const char* fmt, unsigned long long a = 0, unsigned long long b = 0, const char* s = "") {
  char line[512];
  snprintf(line, sizeof line, fmt, s, a, b);
  text += line;
}
int launch(const void* f, Dim g, Dim w) {
  std::lock_guard<std::mutex> lk(mu);
  log("launch %s %llu %llu\n", (unsigned long long)g.x * g.y * g.z, (unsigned long long)w.x * w.y * w.z,
      kernels[f].c_str());
  // A launch holds fewer than 2^32 work-items in each dimension.
  return (uint64_t)g.x * w.x >= (1ull << 32) || (uint64_t)g.y * w.y >= (1ull << 32) ? 9 : 0;
}
thread_local int last_error = 0;
}  // namespace

extern "C" {
// What the test sees and sets: the log so far (then empty), the bytes held, the bytes
// there are, whether events have completed, and the device's compute units.
const char* fake_log() {
  static std::string out;
  std::lock_guard<std::mutex> lk(mu);
  out.swap(text);
  text.clear();
  return out.c_str();
}
size_t fake_used() { return used; }
void fake_limit(size_t n) { limit = n; }
void fake_events(int done) { events_done = done; }
void fake_cus(int n) { cus = n; }

void** __hipRegisterFatBinary(const void*) {
  static void* handle;
  return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, Dim*, Dim*, int*) {
  kernels[f] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim g, Dim w, size_t lds, void* s) {
  cfg_grid = g;
  cfg_block = w;
  cfg_lds = lds;
  cfg_stream = s;
  return 0;
}
int __hipPopCallConfiguration(Dim* g, Dim* w, size_t* lds, void** s) {
  *g = cfg_grid;
  *w = cfg_block;
  *lds = cfg_lds;
  *s = cfg_stream;
  return 0;
}
int hipLaunchKernel(const void* f, Dim g, Dim w, void**, size_t, void*) { return last_error = launch(f, g, w); }
int hipExtLaunchKernel(const void* f, Dim g, Dim w, void**, size_t, void*, void*, void*, int) {
  return last_error = launch(f, g, w);
}
int hipGetLastError() {
  const int e = last_error;
  last_error = 0;
  return e;
}
const char* hipGetErrorString(int) { return "fake error"; }
int hipGetDevice(int* d) {
  *d = 0;
  return 0;
}
int hipSetDevice(int) { return 0; }
int hipDeviceGetAttribute(int* v, int, int) {
  *v = cus;
  return 0;
}
int hipDeviceSynchronize() { return 0; }
int hipMalloc(void** p, size_t n) {
  std::lock_guard<std::mutex> lk(mu);
  if (used + n > limit) return last_error = 2;
  *p = (void*)next_block;
  blocks[next_block] = n;
  next_block += (n + 0xfffff) & ~(size_t)0xfffff;
  used += n;
  log("malloc%s %llu\n", n);
  return 0;
}
int hipFree(void* p) {
  std::lock_guard<std::mutex> lk(mu);
  auto it = blocks.find((uintptr_t)p);
  if (it == blocks.end()) return 1;
  used -= it->second;
  blocks.erase(it);
  return 0;
}
int hipMemset(void*, int, size_t n) {
  std::lock_guard<std::mutex> lk(mu);
  log("memset%s %llu\n", n);
  return 0;
}
int hipMemsetAsync(void* p, int v, size_t n, void*) { return hipMemset(p, v, n); }
int hipMemcpy(void*, const void*, size_t, int) { return 0; }
int hipMemcpyAsync(void*, const void*, size_t, int, void*) { return 0; }
int hipGetSymbolAddress(void** p, const void*) {
  *p = symbols + (n_symbols++ % sizeof symbols);
  return 0;
}
int hipStreamCreate(void** s) {
  *s = symbols;
  return 0;
}
int hipStreamCreateWithFlags(void** s, unsigned) { return hipStreamCreate(s); }
int hipStreamDestroy(void*) { return 0; }
int hipStreamSynchronize(void*) {
  std::lock_guard<std::mutex> lk(mu);
  log("sync%s\n");
  return 0;
}
int hipStreamWaitEvent(void*, void*, unsigned) { return 0; }
int hipEventCreate(void** e) {
  *e = symbols;
  return 0;
}
int hipEventCreateWithFlags(void** e, unsigned) { return hipEventCreate(e); }
int hipEventDestroy(void*) { return 0; }
int hipEventRecord(void*, void*) { return 0; }
int hipEventQuery(void*) { return events_done ? 0 : 600; }
int hipEventSynchronize(void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*) {
  *ms = 1.0f;
  return 0;
}
}
