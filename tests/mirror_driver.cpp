// nlr_api.cpp against a HIP runtime of its own, on the CPU: the functions below take the place of
// the runtime's (this executable's symbols come first) and run no kernel.  They note when a launch
// will write a context's pinned mirror, and fail the check if that memory is freed before the
// stream has been waited for, or if a call that does not wait launches such a write at all.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

#include "nlr_internal.hpp"

static std::map<const void*, std::string>& names() {  // (filled before this file's own initialisers run)
  static auto* m = new std::map<const void*, std::string>;
  return *m;
}
static int g_fails = 0, g_fail_sync = 0;
static bool g_pending = false;  // a launched kernel has yet to write pinned memory
static long g_writes = 0;
static struct { dim3 grid, block; size_t lds; hipStream_t st; } g_call;
static void check(bool ok, const char* what) {
  if (ok) return;
  std::printf("FAIL %s\n", what);
  ++g_fails;
}

extern "C" {
void** __hipRegisterFatBinary(const void*) { return reinterpret_cast<void**>(&g_call); }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  names()[f] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t l, hipStream_t s) {
  g_call = {g, b, l, s};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* l, hipStream_t* s) {
  *g = g_call.grid;
  *b = g_call.block;
  *l = g_call.lds;
  *s = g_call.st;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void** args, size_t, hipStream_t) {
  if (names()[f].find("k_ctl_a") != std::string::npos) {  // (Geometry, Bufs, StepArgs, int finish, ...)
    const nlr::Bufs* b = static_cast<const nlr::Bufs*>(args[1]);
    if (*static_cast<const int*>(args[3]) && b->mirror) {
      g_pending = true;
      ++g_writes;
    }
  }
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void* s) { *p = const_cast<void*>(s); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = std::calloc(1, n); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipHostFree(void* p) {
  check(!g_pending, "pinned memory freed while a launched kernel has yet to write it");
  std::free(p);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void*, size_t n, hipMemcpyKind k, hipStream_t) {
  if (k == hipMemcpyDeviceToHost) std::memset(d, 0, n);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) {
  if (g_fail_sync > 0) {
    --g_fail_sync;
    return hipErrorUnknown;
  }
  g_pending = false;
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = reinterpret_cast<hipStream_t>(&g_call); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) { *g = reinterpret_cast<hipGraph_t>(&g_call); return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  *e = reinterpret_cast<hipGraphExec_t>(&g_call);
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = reinterpret_cast<hipEvent_t>(&g_call); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0.f; return hipSuccess; }
}

static nlr_ctx* open_ctx(int64_t n, int32_t d, int32_t r, uint32_t flags) {
  const nlr_params prm = {0.01, 1.0, 1e-4, 1e-4, 0, 0};
  void* fake = reinterpret_cast<void*>((uintptr_t)1 << 20);  // no kernel runs: never dereferenced
  nlr_ctx* c = nullptr;
  const nlr_status s = nlr_init(&c, (float*)fake, n, d, 4, r, (float*)fake, (float*)fake, &prm, flags, fake,
                                nlr_workspace_bytes(n, d, r), nullptr);
  check(s == NLR_OK && c, "nlr_init");
  return c;
}

int main() {
  const struct { int32_t d, r; uint32_t flags; } forms[] = {
      {64, 16, NLR_INIT_SPLIT_F16}, {64, 32, 0}, {51, 13, 0}, {200, 300, 0}, {768, 256, NLR_INIT_SPLIT_F16}};
  for (auto& f : forms) {
    nlr_iter_stats st;
    int32_t done = 0;
    nlr_ctx* c = open_ctx(5000, f.d, f.r, f.flags);
    g_writes = 0;
    check(nlr_step(c, nullptr) == NLR_OK && nlr_step(c, nullptr) == NLR_OK, "nlr_step without a record");
    check(g_writes == 0, "a step that does not wait writes the mirror");
    nlr_destroy(c);
    c = open_ctx(5000, f.d, f.r, f.flags);
    g_writes = 0;
    check(nlr_step(c, &st) == NLR_OK && !g_pending && g_writes == 1, "nlr_step with its record");
    check(nlr_run(c, 40, &done, &st) == NLR_OK && !g_pending && g_writes == 2, "nlr_run");
    check(nlr_step(c, nullptr) == NLR_OK && g_writes == 2, "nlr_step without a record, after a run");
    nlr_destroy(c);
    c = open_ctx(5000, f.d, f.r, f.flags);
    g_fail_sync = 1;  // the wait fails: the write may still be outstanding
    check(nlr_step(c, &st) == NLR_EHIP && g_pending, "nlr_step whose wait fails");
    nlr_destroy(c);
    g_pending = false;
  }
  std::printf(g_fails ? "%d checks failed\n" : "all checks passed\n", g_fails);
  return g_fails ? 1 : 0;
}
