// A stand-in for the HIP runtime and the kernels, for tests of the library's host code on machines
// without a GPU: device memory is host memory, launches do nothing, an event completes a settable
// time after it is waited for.  It counts what is alive, and can make an allocation or a thread
// start fail.
#include "fake_hip.h"

#include <dlfcn.h>
#include <errno.h>
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <pthread.h>
#include <sched.h>
#include <stdlib.h>
#include <string.h>
#include <time.h>

#include <atomic>
#include <new>

#include "hs_kernels.h"

namespace fake {
std::atomic<long> live_objects{0}, live_blocks{0}, live_threads{0};
std::atomic<long> event_wait_ns{0};
std::atomic<long> mask_queries{0};
std::atomic<long> blocks_until_failure{-1}, threads_until_failure{-1};
std::atomic<bool> fail_block_after_thread_start{false};
static thread_local bool fail_next_block = false;
hs::ConvParams conv_launches[kMaxConvLaunches];
std::atomic<int> n_conv_launches{0};
void* launch_streams[kMaxLaunches];
std::atomic<int> n_launches{0};
thread_local int device = 0;
uint64_t overlay_drawn = 500;
int32_t overlay_maxima = 300;
static hipError_t launched(hipStream_t s) {
  const int n = n_launches++;
  if (n < kMaxLaunches) launch_streams[n] = s;
  return hipSuccess;
}
void reset_failures() {
  blocks_until_failure = threads_until_failure = -1;
  fail_block_after_thread_start = false;
  fail_next_block = false;
}
}  // namespace fake
using namespace fake;

// ---- allocations and thread starts ---------------------------------------------------------------
static void* take_block(size_t n) {
  if (fail_next_block) { fail_next_block = false; throw std::bad_alloc(); }
  if (blocks_until_failure >= 0 && blocks_until_failure.fetch_sub(1) == 0) throw std::bad_alloc();
  void* p = malloc(n ? n : 1);
  if (!p) throw std::bad_alloc();
  ++live_blocks;
  return p;
}
static void give_block(void* p) {
  if (p) --live_blocks;
  free(p);
}
void* operator new(size_t n) { return take_block(n); }
void* operator new[](size_t n) { return take_block(n); }
void* operator new(size_t n, const std::nothrow_t&) noexcept {
  try { return take_block(n); } catch (const std::bad_alloc&) { return nullptr; }
}
void operator delete(void* p) noexcept { give_block(p); }
void operator delete[](void* p) noexcept { give_block(p); }
void operator delete(void* p, size_t) noexcept { give_block(p); }
void operator delete[](void* p, size_t) noexcept { give_block(p); }
void operator delete(void* p, const std::nothrow_t&) noexcept { give_block(p); }

struct Start { void* (*f)(void*); void* x; };
static void* counted(void* p) {
  const Start s = *(Start*)p;
  free(p);
  void* r = s.f(s.x);
  --live_threads;
  return r;
}
extern "C" int sched_getaffinity(pid_t pid, size_t size, cpu_set_t* set) noexcept {
  using Fn = int (*)(pid_t, size_t, cpu_set_t*);
  static Fn real = (Fn)dlsym(RTLD_NEXT, "sched_getaffinity");
  ++fake::mask_queries;
  return real(pid, size, set);
}

extern "C" int pthread_create(pthread_t* t, const pthread_attr_t* a, void* (*f)(void*), void* x) {
  using Fn = int (*)(pthread_t*, const pthread_attr_t*, void* (*)(void*), void*);
  static Fn real = (Fn)dlsym(RTLD_NEXT, "pthread_create");
  if (threads_until_failure >= 0 && threads_until_failure.fetch_sub(1) == 0) return EAGAIN;
  Start* s = (Start*)malloc(sizeof(Start));
  *s = Start{f, x};
  ++live_threads;
  const int rc = real(t, a, counted, s);
  if (rc == 0 && fail_block_after_thread_start.exchange(false)) fail_next_block = true;
  return rc;
}

// ---- HIP runtime -----------------------------------------------------------------------------------
template <class T> static hipError_t make(T* out) {
  *out = (T)malloc(1);
  ++live_objects;
  return hipSuccess;
}
template <class T> static hipError_t drop(T x) {
  free((void*)x);
  --live_objects;
  return hipSuccess;
}
extern "C" {
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipSetDevice(int d) { fake::device = d; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = fake::device; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  memset(p, 0, sizeof(*p));
  strcpy(p->gcnArchName, "gfx950");
  p->multiProcessorCount = 256;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 100000; return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "fake"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemset(void* d, int v, size_t n) { memset(d, v, n); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  *p = malloc(n);
  ++live_objects;
  return hipSuccess;
}
hipError_t hipHostFree(void* p) { return drop(p); }
hipError_t hipEventCreate(hipEvent_t* e) { return make(e); }
hipError_t hipEventDestroy(hipEvent_t e) { return drop(e); }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) {
  const long ns = event_wait_ns;
  timespec t = {ns / 1000000000, ns % 1000000000};
  if (ns) nanosleep(&t, nullptr);
  return hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0.001f; return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { return make(s); }
hipError_t hipExtStreamCreateWithCUMask(hipStream_t* s, uint32_t, const uint32_t*) { return make(s); }
hipError_t hipStreamDestroy(hipStream_t s) { return drop(s); }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t s) { return launched(s); }
hipError_t hipExtLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t s, hipEvent_t, hipEvent_t, int) {
  return launched(s);
}
hipError_t hipGraphCreate(hipGraph_t* g, unsigned) { return make(g); }
hipError_t hipGraphDestroy(hipGraph_t g) { return drop(g); }
hipError_t hipGraphAddKernelNode(hipGraphNode_t* n, hipGraph_t, const hipGraphNode_t*, size_t, const hipKernelNodeParams*) {
  *n = nullptr;
  return hipSuccess;
}
hipError_t hipGraphAddEventRecordNode(hipGraphNode_t* n, hipGraph_t, const hipGraphNode_t*, size_t, hipEvent_t) {
  *n = nullptr;
  return hipSuccess;
}
hipError_t hipGraphAddEventWaitNode(hipGraphNode_t* n, hipGraph_t, const hipGraphNode_t*, size_t, hipEvent_t) {
  *n = nullptr;
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) { return make(e); }
hipError_t hipGraphExecDestroy(hipGraphExec_t e) { return drop(e); }
hipError_t hipGraphExecKernelNodeSetParams(hipGraphExec_t, hipGraphNode_t, const hipKernelNodeParams*) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
}

// ---- kernels ---------------------------------------------------------------------------------------
namespace hs {
static int some_kernel;
static KernelDesc some() { return KernelDesc{&some_kernel, dim3(1), dim3(64), 0}; }
KernelDesc describe(const ResizeParams&) { return some(); }
KernelDesc describe(const ConvParams& p) {
  if (p.wt_frag && fake::n_conv_launches < fake::kMaxConvLaunches) fake::conv_launches[fake::n_conv_launches++] = p;
  return some();
}
KernelDesc describe(const TinyFrameParams& p) {   // a launch of the small network as well
  ConvParams c{};
  c.variant = CONV_TINY_NET;
  c.wt_frag = p.wt_frag;
  return describe(c);
}
KernelDesc describe(const LstmEpilogueParams&) { return some(); }
KernelDesc describe(const StemPoolParams&) { return some(); }
KernelDesc describe(const PostParams&) { return some(); }
KernelDesc describe(const OverlayParams& p) {
  for (int l = 0; l < p.n_layers; ++l) {
    const OverlayLayer& L = p.layer[l];
    if (L.stamps) *L.stamps = StageStamps{100000, 200000, 0, 200000 + fake::overlay_drawn};
    for (int j = 0; L.rec && j < p.batch; ++j) L.rec[j].ticks[j % 8] = fake::overlay_maxima;
  }
  return some();
}
hipError_t static_scratch_address(void** p, size_t* n) {
  static char scratch[256];
  *p = scratch;
  *n = sizeof(scratch);
  return hipSuccess;
}
void launch_fill_zero(void*, size_t, hipStream_t) {}
void launch_copy(void*, const void*, size_t, hipStream_t) {}
}  // namespace hs
