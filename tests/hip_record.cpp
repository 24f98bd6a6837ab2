// A HIP runtime for tests on the CPU: memory is host memory, launches, events and stream waits are only
// written down, and setting a kernel's LDS limit can be made to fail.  Linked with the library's objects in
// place of the real runtime, it shows what the host code queues, in which order and on which stream.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

namespace {
std::map<const void*, std::string> g_names;
std::string g_log, g_fail;
dim3 g_grid, g_block;
size_t g_lds;
hipStream_t g_stream;
uintptr_t g_next = 0x1000;

void line(const char* fmt, const char* name, long long a, long long b, long long c = 0, long long d = 0,
          long long e = 0) {
  char buf[1024];
  std::snprintf(buf, sizeof(buf), fmt, name, a, b, c, d, e);
  g_log += buf;
}
template <typename T>
T handle() {
  return reinterpret_cast<T>(g_next += 0x10);
}
}  // namespace

extern "C" {
const char* rec_log() { return g_log.c_str(); }
void rec_clear() { g_log.clear(); }
// LDS limits of kernels whose name contains this cannot be set (empty: all can)
void rec_fail_attribute(const char* part) { g_fail = part; }

void** __hipRegisterFatBinary(const void*) { return handle<void**>(); }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  g_names[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s) {
  g_grid = g;
  g_block = b;
  g_lds = lds;
  g_stream = s;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, hipStream_t* s) {
  *g = g_grid;
  *b = g_block;
  *lds = g_lds;
  *s = g_stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void**, size_t lds, hipStream_t s) {
  line("launch %s %lld %lld %lld %lld %lld\n", g_names[f].c_str(), (long long)s, g.x, b.x, (long long)lds, g.z);
  return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void* f, hipFuncAttribute, int) {
  return !g_fail.empty() && g_names[f].find(g_fail) != std::string::npos ? hipErrorInvalidValue : hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
  *n = 1;
  return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) {
  *p = std::calloc(1, n ? n : 1);
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void* p) {
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
  *v = 256;
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "recorded"; }
hipError_t hipGetSymbolAddress(void** p, const void*) {
  static void* mem = std::calloc(1, 16 << 20);
  *p = mem;
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = handle<hipStream_t>();
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  line("wait %s%lld %lld\n", "", (long long)s, (long long)e);
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) {
  *e = handle<hipEvent_t>();
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  line("record %s%lld %lld\n", "", (long long)s, (long long)e);
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 1.0f;
  return hipSuccess;
}
}
