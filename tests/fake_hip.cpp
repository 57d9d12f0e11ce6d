// A HIP runtime that runs nothing and writes down what it is asked, so that the
// host side of libpfmm (what is allocated, freed, ordered and launched) can be
// checked without a GPU.  Device addresses are opaque; launches do nothing; a
// launch or an allocation can be made to fail.
#include <stdint.h>
#include <string.h>

#include <map>
#include <mutex>
#include <string>

struct dim3_ {
  uint32_t x, y, z;
};

namespace {
std::mutex mu;
std::string text;                          // the log, a line a call
std::map<const void*, std::string> names;  // host stub -> kernel
std::map<uintptr_t, size_t> live;          // allocations
uintptr_t next_address = 1ull << 40, next_handle = 1 << 20;
size_t used = 0, total = 288ull << 30;
int fail_launches = 0, pending = 0;
const void* captured = nullptr;  // the stream being captured
struct {
  dim3_ g, b;
  size_t sh;
  void* st;
} call;

void say(const std::string& s) {
  std::lock_guard<std::mutex> lk(mu);
  text += s + "\n";
}
std::string hex(const void* p) { return std::to_string((uintptr_t)p); }
int handle(void** out, const char* what) {
  *out = (void*)(next_handle += 64);
  say(std::string(what) + " " + hex(*out));
  return 0;
}
}  // namespace

extern "C" {
// --- for the test ---
const char* fake_log() {  // the lines since the last call
  static std::string out;
  std::lock_guard<std::mutex> lk(mu);
  out.swap(text);
  text.clear();
  return out.c_str();
}
void fake_fail_launches(int on) { fail_launches = on; }
void fake_capture(const void* stream) { captured = stream; }
void fake_total(size_t bytes) { total = bytes; }
size_t fake_used() { return used; }

// --- the runtime ---
void** __hipRegisterFatBinary(const void*) {
  static void* module = nullptr;
  return &module;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*,
                           void*, int*) {
  names[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(dim3_ g, dim3_ b, size_t sh, void* st) {
  call = {g, b, sh, st};
  return 0;
}
int __hipPopCallConfiguration(dim3_* g, dim3_* b, size_t* sh, void** st) {
  *g = call.g;
  *b = call.b;
  *sh = call.sh;
  *st = call.st;
  return 0;
}
int hipLaunchKernel(const void* f, dim3_, dim3_, void**, size_t, void* st) {
  if (fail_launches) return pending = 719;
  say("launch " + names[f] + " " + hex(st));
  return 0;
}
int hipGetLastError() {
  const int e = pending;
  pending = 0;
  return e;
}
const char* hipGetErrorString(int) { return "made to fail"; }
int hipMalloc(void** p, size_t n) {
  if (used + n > total) return pending = 2;
  used += n;
  *p = (void*)next_address;
  live[next_address] = n;
  next_address += (n + 4095) / 4096 * 4096;
  say("malloc " + hex(*p) + " " + std::to_string(n));
  return 0;
}
int hipFree(void* p) {
  if (!p) return 0;
  auto it = live.find((uintptr_t)p);
  if (it == live.end()) return pending = 1;
  used -= it->second;
  live.erase(it);
  say("free " + hex(p));
  return 0;
}
int hipMemGetInfo(size_t* free_bytes, size_t* all) {
  *free_bytes = total - used;
  *all = total;
  return 0;
}
int hipMemcpy(void* dst, const void*, size_t n, int kind) {
  if (kind == 2) memset(dst, 0, n);  // to the host
  return 0;
}
int hipMemcpyAsync(void* dst, const void* src, size_t n, int kind, void*) { return hipMemcpy(dst, src, n, kind); }
int hipMemset(void*, int, size_t) { return 0; }
int hipMemsetAsync(void*, int, size_t, void*) { return 0; }
int hipGetDevice(int* d) {
  *d = 0;
  return 0;
}
int hipDeviceGetAttribute(int* v, int, int) {
  *v = 256;
  return 0;
}
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
  *n = 1;
  return 0;
}
int hipDeviceSynchronize() {
  say("device-sync");
  return 0;
}
int hipStreamSynchronize(void* st) {
  say("sync " + hex(st));
  return 0;
}
int hipStreamCreateWithFlags(void** st, unsigned) { return handle(st, "stream"); }
int hipStreamDestroy(void*) { return 0; }
int hipStreamWaitEvent(void* st, void* e, unsigned) {
  say("wait " + hex(st) + " " + hex(e));
  return 0;
}
int hipStreamIsCapturing(void* st, int* status) {
  *status = captured && st == captured ? 1 : 0;
  return 0;
}
int hipEventCreate(void** e) { return handle(e, "event"); }
int hipEventCreateWithFlags(void** e, unsigned) { return handle(e, "event"); }
int hipEventDestroy(void*) { return 0; }
int hipEventRecord(void* e, void* st) {
  say("record " + hex(e) + " " + hex(st));
  return 0;
}
int hipEventSynchronize(void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*) {
  *ms = 1.0f;
  return 0;
}
}
