// A HIP runtime for host tests: memory is host memory, kernels do nothing, and the calls that order work
// (streams, events, graphs) are logged.  stub_fail makes the nth coming call of a function fail.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <string>

static std::string g_log, g_fail;
static int g_nth = 0, g_ready = 1;
static uintptr_t g_next = 0x10000;

static int step(const char* name, const void* a = nullptr, const void* b = nullptr) {
  const bool bad = g_fail == name && g_nth > 0 && --g_nth == 0;
  char line[128];
  snprintf(line, sizeof(line), "%s %lx %lx %d\n", name, (unsigned long)(uintptr_t)a, (unsigned long)(uintptr_t)b, bad ? 1 : 0);
  g_log += line;
  return bad ? 999 : 0;
}
static void* handle() { return (void*)(g_next += 16); }
static int alloc(void** p, size_t n) { return (*p = calloc(n ? n : 1, 1)) ? 0 : 2; }

extern "C" {
const char* stub_log() { return g_log.c_str(); }
void stub_clear() { g_log.clear(); }
void stub_ready(int ready) { g_ready = ready; }   // whether recorded events are done
void stub_fail(const char* name, int nth) { g_fail = name; g_nth = nth; }

int hipGetDeviceCount(int* n) { *n = 1; return 0; }
int hipSetDevice(int) { return 0; }
int hipDeviceGetAttribute(int* v, int, int) { *v = 256; return 0; }
int hipDeviceSynchronize() { return 0; }
int hipGetLastError() { return 0; }
int hipGetSymbolAddress(void** p, const void*) { return alloc(p, 1 << 16); }
int hipMalloc(void** p, size_t n) { return alloc(p, n); }
int hipFree(void* p) { free(p); return 0; }
int hipMemset(void* p, int v, size_t n) { memset(p, v, n); return 0; }
int hipMemcpy(void* d, const void* s, size_t n, int) { memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void*) { memcpy(d, s, n); return 0; }
int __hipPushCallConfiguration(uint64_t, uint32_t, uint64_t, uint32_t, size_t, void*) { return 0; }
int __hipPopCallConfiguration(void* g, void* b, size_t* m, void** s) {
  memset(g, 0, 12);
  memset(b, 0, 12);
  *m = 0;
  *s = nullptr;
  return 0;
}
int hipLaunchKernel(const void*, uint64_t, uint32_t, uint64_t, uint32_t, void**, size_t, void*) { return 0; }
int hipExtLaunchKernel(const void*, uint64_t, uint32_t, uint64_t, uint32_t, void**, size_t, void*, void*, void*, int) { return 0; }
int hipStreamCreateWithFlags(void** s, unsigned) { return *s = handle(), step("create", *s); }
int hipStreamDestroy(void* s) { return step("destroy", s); }
int hipStreamSynchronize(void* s) { return step("sync", s); }
int hipStreamWaitEvent(void* s, void* e, unsigned) { return step("wait", s, e); }
int hipStreamIsCapturing(void*, int* st) { *st = 0; return 0; }
int hipStreamBeginCapture(void*, int) { return 0; }
int hipStreamEndCapture(void*, void** g) { *g = handle(); return 0; }
int hipGraphInstantiate(void** x, void*, void*, void*, size_t) { *x = handle(); return 0; }
int hipGraphLaunch(void* x, void* s) { return step("launch", s, x); }
int hipGraphExecDestroy(void*) { return 0; }
int hipGraphDestroy(void*) { return 0; }
int hipEventCreateWithFlags(void** e, unsigned) { *e = handle(); return 0; }
int hipEventQuery(void*) { return g_ready ? 0 : 600; }
int hipEventDestroy(void*) { return 0; }
int hipEventRecord(void* e, void* s) { return step("record", s, e); }
}
