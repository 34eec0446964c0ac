// A device that is not there: the HIP runtime calls that the library makes, for tests of its host side without a GPU.  Memory is
// counted against a budget and never touched, launches are checked against the limits of the runtime and recorded.
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>

#include <map>
#include <mutex>
#include <string>

struct dim3 {
  uint32_t x, y, z;
};
enum { kSuccess = 0, kOutOfMemory = 2, kInvalidConfiguration = 9 };

static size_t g_budget = ~(size_t)0, g_used = 0, g_peak = 0;
static int g_mallocs = 0, g_capturing = 0;
static uintptr_t g_next = (uintptr_t)1 << 40;
static std::map<uintptr_t, size_t> g_live;
static std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> m;
  return m;
}
static std::string g_log;
static thread_local dim3 g_grid, g_block;
static thread_local void* g_stream;
static std::mutex g_mutex;
static std::string g_watched;
static int g_argument = 0;
static uintptr_t g_value = 0;

extern "C" {
// ---- what a test sees and sets
void fake_budget(size_t bytes) { g_budget = bytes; }
size_t fake_used() { return g_used; }
size_t fake_peak() { return g_peak; }
int fake_mallocs() { return g_mallocs; }
void fake_capturing(int on) { g_capturing = on; }  // every stream
const char* fake_launches() {  // since the last call, "name gx gy gz bx\n" each
  static std::string out;
  out.swap(g_log);
  g_log.clear();
  return out.c_str();
}

// from now on, pointer argument `i` of the last launch of a kernel whose name contains `part`
void fake_watch(const char* part, int i) {
  g_watched = part;
  g_argument = i;
}
uintptr_t fake_argument() { return g_value; }

// ---- memory
int hipMalloc(void** p, size_t n) {
  std::lock_guard<std::mutex> lock(g_mutex);
  ++g_mallocs;
  if (g_used + n > g_budget) return kOutOfMemory;
  *p = (void*)g_next;
  g_live[g_next] = n;
  g_next += (n + 4095) / 4096 * 4096;
  g_used += n;
  if (g_used > g_peak) g_peak = g_used;
  return kSuccess;
}
int hipFree(void* p) {
  std::lock_guard<std::mutex> lock(g_mutex);
  auto it = g_live.find((uintptr_t)p);
  if (it != g_live.end()) {
    g_used -= it->second;
    g_live.erase(it);
  }
  return kSuccess;
}
int hipMemset(void*, int, size_t) { return kSuccess; }
int hipMemcpy(void*, const void*, size_t, int) { return kSuccess; }
int hipGetSymbolAddress(void** p, const void*) {
  *p = (void*)((uintptr_t)1 << 39);
  return kSuccess;
}

// ---- device, streams, events
int hipThreadExchangeStreamCaptureMode(int*) { return kSuccess; }
int hipSetDevice(int) { return kSuccess; }
int hipGetDevice(int* d) {
  *d = 0;
  return kSuccess;
}
int hipDeviceGetAttribute(int* v, int, int) {
  *v = 256;
  return kSuccess;
}
int hipDeviceSynchronize() { return kSuccess; }
int hipStreamSynchronize(void*) { return kSuccess; }
int hipStreamCreateWithFlags(void** s, unsigned) {
  static uintptr_t next = 16;
  *s = (void*)(next += 16);
  return kSuccess;
}
int hipStreamDestroy(void*) { return kSuccess; }
int hipStreamIsCapturing(void*, int* status) {
  *status = g_capturing;
  return kSuccess;
}
int hipStreamWaitEvent(void*, void*, unsigned) { return kSuccess; }
int hipEventCreate(void** e) { return hipStreamCreateWithFlags(e, 0); }
int hipEventCreateWithFlags(void** e, unsigned) { return hipStreamCreateWithFlags(e, 0); }
int hipEventDestroy(void*) { return kSuccess; }
int hipEventRecord(void*, void*) { return kSuccess; }
int hipEventSynchronize(void*) { return kSuccess; }
int hipEventElapsedTime(float* ms, void*, void*) {
  *ms = 0.0f;
  return kSuccess;
}

// ---- kernels
void** __hipRegisterFatBinary(const void*) {
  static void* handle = nullptr;
  return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  names()[host] = name;
}
int hipFuncSetAttribute(const void*, int, int) { return kSuccess; }
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t, void* stream) {
  g_grid = grid;
  g_block = block;
  g_stream = stream;
  return kSuccess;
}
int __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, void** stream) {
  *grid = g_grid;
  *block = g_block;
  *lds = 0;
  *stream = g_stream;
  return kSuccess;
}
static int g_launch_error = 0;
int hipGetLastError() {
  const int e = g_launch_error;
  g_launch_error = kSuccess;
  return e;
}
int hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t, void*) {
  char line[512];
  std::lock_guard<std::mutex> lock(g_mutex);
  if (!g_watched.empty() && names()[f].find(g_watched) != std::string::npos) g_value = *(uintptr_t*)args[g_argument];
  const bool bad = grid.x == 0 || grid.y == 0 || grid.z == 0 || grid.y > 65535 || grid.z > 65535 || block.x > 1024 ||
                   (uint64_t)grid.x * block.x > 0xffffffffu;  // the runtime counts work-items per dimension in 32 bits
  snprintf(line, sizeof line, "%s%s %u %u %u %u\n", bad ? "REFUSED " : "", names()[f].c_str(), grid.x, grid.y, grid.z, block.x);
  g_log += line;
  if (bad) g_launch_error = kInvalidConfiguration;
  return bad ? kInvalidConfiguration : kSuccess;
}
}
