// A HIP runtime without a GPU, for tests of the library's host side: two
// devices whose memory is host memory, copies made at once, launches written to a
// log instead of run, and the runtime's rules that the tests look at: an event is
// recorded on streams of its own device only, nothing synchronizes while a
// stream is captured, an event whose stream is gone cannot be waited for, a grid
// has fewer than 2^32 threads in x.  Preloaded before libamdhip64 (see fake_hip.py).
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <string>

namespace {
struct Event {
  int dev;
  hipStream_t on;  // recorded on last
};
struct Stream {
  int dev;
};
int g_dev = 0;
bool g_capture = false;
hipError_t g_last = hipSuccess;
std::string g_log;
std::map<const void*, std::string> g_names;
std::map<const void*, void*> g_symbols;
std::map<void*, size_t> g_allocs;
std::set<hipStream_t> g_gone;
size_t g_held = 0, g_peak = 0, g_limit = ~(size_t)0;
dim3 g_grid, g_block;
hipStream_t g_stream;

hipError_t fail(hipError_t e) { return g_last = e; }
hipError_t sync_allowed() { return g_capture ? fail(hipErrorStreamCaptureUnsupported) : hipSuccess; }
int device_of(hipStream_t s) { return s ? reinterpret_cast<Stream*>(s)->dev : g_dev; }
}  // namespace

extern "C" {
// ---- the tests' side
void fake_set_device(int d) { g_dev = d; }
void fake_capture(int on) { g_capture = on != 0; }
void fake_limit(size_t bytes) { g_limit = bytes; }
size_t fake_peak(int reset) {
  const size_t p = g_peak;
  if (reset) g_peak = g_held;
  return p;
}
const char* fake_log(int clear) {
  static std::string out;
  out = g_log;
  if (clear) g_log.clear();
  return out.c_str();
}

// ---- registration and launches
void** __hipRegisterFatBinary(const void*) {
  static void* one;
  return &one;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*,
                           void*, void*, int*) {
  g_names[host] = name;
}
void __hipRegisterVar(void**, void* var, char*, char*, int, size_t size, int, int) {
  g_symbols[var] = calloc(1, size);
}
hipError_t hipGetSymbolAddress(void** p, const void* symbol) {
  *p = g_symbols[symbol];
  return *p ? hipSuccess : fail(hipErrorInvalidSymbol);
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t, hipStream_t st) {
  g_grid = grid;
  g_block = block;
  g_stream = st;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* st) {
  *grid = g_grid;
  *block = g_block;
  *shared = 0;
  *st = g_stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void**, size_t, hipStream_t) {
  if ((unsigned long long)grid.x * block.x >= 1ull << 32 || grid.x == 0 || grid.y == 0)
    return fail(hipErrorInvalidConfiguration);
  char line[64];
  snprintf(line, sizeof line, " %u %u\n", grid.x, grid.y);
  g_log += g_names[f] + line;
  return hipSuccess;
}

// ---- memory
hipError_t hipMalloc(void** p, size_t n) {
  if (g_held + n > g_limit) return fail(hipErrorOutOfMemory);
  *p = malloc(n);
  if (!*p) return fail(hipErrorOutOfMemory);
  g_allocs[*p] = n;
  g_held += n;
  if (g_held > g_peak) g_peak = g_held;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  if (p) {
    g_held -= g_allocs[p];
    g_allocs.erase(p);
  }
  free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  *p = malloc(n);
  return *p ? hipSuccess : fail(hipErrorOutOfMemory);
}
hipError_t hipHostFree(void* p) {
  free(p);
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  const hipError_t e = sync_allowed();
  if (e == hipSuccess) memcpy(d, s, n);
  return e;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  memcpy(d, s, n);
  return hipSuccess;
}

// ---- streams and events
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = reinterpret_cast<hipStream_t>(new Stream{g_dev});
  return hipSuccess;
}
hipError_t hipStreamCreate(hipStream_t* s) { return hipStreamCreateWithFlags(s, 0); }
hipError_t hipStreamDestroy(hipStream_t s) {
  g_gone.insert(s);  // kept, so that no other stream gets its address
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return sync_allowed(); }
hipError_t hipDeviceSynchronize() { return sync_allowed(); }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* c) {
  *c = g_capture ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
// What the runtime has returned for events whose stream was destroyed.
static hipError_t event_stream(hipEvent_t e) {
  return g_gone.count(reinterpret_cast<Event*>(e)->on) ? fail(hipErrorCapturedEvent) : hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t e, unsigned) { return event_stream(e); }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  *e = reinterpret_cast<hipEvent_t>(new Event{g_dev, nullptr});
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) {
  delete reinterpret_cast<Event*>(e);
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  if (reinterpret_cast<Event*>(e)->dev != device_of(s)) return fail(hipErrorInvalidHandle);
  reinterpret_cast<Event*>(e)->on = s;
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
  const hipError_t r = event_stream(e);
  return r == hipSuccess ? sync_allowed() : r;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 0.f;
  return hipSuccess;
}

// ---- devices and errors
hipError_t hipGetDeviceCount(int* n) {
  *n = 2;
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
  *d = g_dev;
  return hipSuccess;
}
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int) {  // the header maps the name
  memset(p, 0, sizeof *p);
  strcpy(p->gcnArchName, "gfx950");
  return hipSuccess;
}
hipError_t hipGetLastError() {
  const hipError_t e = g_last;
  g_last = hipSuccess;
  return e;
}
const char* hipGetErrorString(hipError_t e) {
  static char s[32];
  snprintf(s, sizeof s, "fake HIP error %d", (int)e);
  return s;
}
}
