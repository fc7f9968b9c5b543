// What the library's calls ask of the HIP runtime, without a device: the functions below stand in front of the runtime's own
// (a program's symbols come before those of its libraries). Prints one line per call, the events in order:
//   A alloc  a stream-ordered alloc  L launch  f stream-ordered free, each with the stream's name (0 default, P hipStreamPerThread, 1, 2 ...)
#include <hip/hip_runtime.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <string>
#include <thread>
#include <utility>
#include <vector>

#include "../../include/mlt_diag.h"

static std::string g_events;
static bool g_capturing = false;
static std::string name(hipStream_t s) { return s == hipStreamPerThread ? "P" : std::to_string((uintptr_t)s >> 12); }
static void event(const char* what, hipStream_t s) { g_events += std::string(g_events.empty() ? "" : " ") + what + name(s); }

extern "C" {
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  memset(p, 0, sizeof *p);
  strcpy(p->gcnArchName, "gfx950:sramecc+:xnack-");
  p->multiProcessorCount = 256;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
  *v = a == hipDeviceAttributeNumberOfXccs ? 8 : 256;
  return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* st) {
  *st = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) { *p = malloc(n); g_events += std::string(g_events.empty() ? "" : " ") + "A"; return hipSuccess; }
hipError_t hipFree(void* p) { free(p); return hipSuccess; }
hipError_t hipMallocAsync(void** p, size_t n, hipStream_t s) { *p = malloc(n); event("a", s); return hipSuccess; }
hipError_t hipFreeAsync(void* p, hipStream_t s) { free(p); event("f", s); return hipSuccess; }
static thread_local struct { dim3 g, b; size_t m; hipStream_t s; } t_conf;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t m, hipStream_t s) { t_conf = {g, b, m, s}; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* m, hipStream_t* s) {
  *g = t_conf.g; *b = t_conf.b; *m = t_conf.m; *s = t_conf.s;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t s) { event("L", s); return hipSuccess; }
}

static void* at(uintptr_t mib) { return (void*)(mib << 20); }   // operands: addresses that nobody follows
static void call(const char* what, void* s) {
  g_events.clear();
  int rc = -99;
  if (!strcmp(what, "gemm")) rc = mlt_gemm(16, 1024, 8192, at(1), 8192, at(2), 8192, 1, at(99), 1024, MLT_BF16, s);
  if (!strcmp(what, "tiles")) rc = mlt_gemm(777, 4096, 14336, at(1), 14336, at(99), 14336, 1, at(999), 4096, MLT_BF16, s);
  if (!strcmp(what, "tall")) rc = mlt_gemm(44, 7296, 11456, at(1), 11456, at(99), 11456, 1, at(999), 7296, MLT_BF16, s);
  if (!strcmp(what, "mha")) rc = mlt_mha_fwd(1, 8, 1, 4096, 128, at(1), at(2), at(99), at(999), 0.1f, 0, MLT_BF16, s);
  if (!strcmp(what, "paged"))
    rc = mlt_paged_attn_decode(1, 8, 128, 16, 256, 256, at(1), at(2), at(99), (const int32_t*)at(500), (const int32_t*)at(501), at(999), 0.1f, MLT_BF16, s);
  if (!strcmp(what, "few"))
    rc = mlt_paged_attn_decode(1, 8, 64, 16, 44, 256, at(1), at(2), at(99), (const int32_t*)at(500), (const int32_t*)at(501), at(999), 0.1f, MLT_BF16, s);
  printf("%d %s: %s\n", rc, mlt_last_kernel(), g_events.c_str());
}

int main() {
  std::vector<std::pair<std::string, std::string>> in;
  char what[16], stream[8];
  while (scanf("%15s %7s", what, stream) == 2) in.emplace_back(what, stream);
  for (size_t i = 0, n; i < in.size(); i += n) {
    const std::string& st = in[i].second;
    for (n = 1; i + n < in.size() && in[i + n].second == st; ++n) {}
    g_capturing = st[0] == 'c';                                 // a stream that records into a graph
    void* s = st[0] == 'P' ? (void*)hipStreamPerThread : g_capturing ? (void*)0x777000 : (void*)((uintptr_t)atoi(st.c_str()) << 12);
    auto calls = [&] { for (size_t k = i; k < i + n; ++k) call(in[k].first.c_str(), s); };
    if (st[0] == 'P') std::thread(calls).join();                // P1 P1 P2: two calls of one thread, one of another
    else calls();
  }
}
