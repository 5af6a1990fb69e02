// A stand-in for the HIP runtime calls libcomet makes: nothing runs on a device;
// every call that allocates, copies, waits or launches is written down in order.
// Loaded with global symbols before libcomet, so that its calls come here.
#include <hip/hip_runtime_api.h>

#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

namespace {
std::string g_log;
std::map<const void*, std::string> g_names;
struct Config {
  dim3 grid, block;
  size_t lds;
  hipStream_t stream;
} g_config;
uintptr_t g_next_stream = 0x5000;

void put(const char* fmt, ...) {
  char b[1024];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(b, sizeof b, fmt, ap);
  va_end(ap);
  g_log += b;
  g_log += '\n';
}
size_t id(hipStream_t s) { return reinterpret_cast<size_t>(s); }
}  // namespace

extern "C" {

const char* record_log() { return g_log.c_str(); }
void record_clear() { g_log.clear(); }

static void* g_module;
void** __hipRegisterFatBinary(const void*) { return &g_module; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*,
                           void*, void*, int*) {
  g_names[f] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s) {
  g_config = {g, b, lds, s};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, hipStream_t* s) {
  *g = g_config.grid;
  *b = g_config.block;
  *lds = g_config.lds;
  *s = g_config.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3, void**, size_t, hipStream_t s) {
  put("launch %zu %s %u %u", id(s), g_names[f].c_str(), g.x, g.y);
  return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "recorded"; }
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
#undef hipGetDeviceProperties
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  memset(p, 0, sizeof *p);
  strcpy(p->gcnArchName, "gfx950");
  p->multiProcessorCount = 256;
  return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) {
  *p = calloc(1, n);
  put("malloc %zu", n);
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  free(p);
  put("free");
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) {
  static void* a = calloc(1, size_t(80) << 20);
  *p = a;
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  memcpy(d, s, n);
  put("memcpy %zu", n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t st) {
  memcpy(d, s, n);
  put("memcpy_async %zu %zu", id(st), n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t st) {
  memset(d, v, n);
  put("memset_async %zu %zu", id(st), n);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
  put("synchronize %zu", id(s));
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = reinterpret_cast<hipStream_t>(g_next_stream++);
  put("stream_create %zu", id(*s));
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
  put("stream_destroy %zu", id(s));
  return hipSuccess;
}
}
