// Beside hip_stub.cpp, for tests/test_host_step.py: a stream under capture by
// the caller, a graph that cannot be instantiated, device memory that is short, and
// records of what lbm_step enqueued (linked with --wrap for the functions hip_stub.cpp defines).
#include <hip/hip_runtime.h>

#include "../../paper_2202_12147_amd/csrc/common.h"

using lbmib::Dev;

namespace {
int g_capturing = 0;        // the caller captures the stream
int g_fail_instantiate = 0; // graphs cannot be instantiated
bool g_own = false;         // inside a capture of the library's own
int g_fail_launch = -1;     // graph launches that still succeed; -1: all
size_t g_malloc_limit = ~size_t(0);  // larger device allocations fail
long g_mallocs = 0, g_frees = 0;
long g_marks = 0, g_steps = 0, g_graph_steps = 0, g_launched = 0;
}  // namespace

extern "C" {
void control(int capturing, int fail_instantiate, int fail_launch) {
  g_capturing = capturing;
  g_fail_instantiate = fail_instantiate;
  g_fail_launch = fail_launch;
}
void limit_malloc(size_t bytes) { g_malloc_limit = bytes; }
void allocations(long out[2]) {
  out[0] = g_mallocs;
  out[1] = g_frees;
}
// Prologue marks launched, steps whose closing launch was made directly, steps
// replayed from graphs; graph launches.
void records(long out[4]) {
  out[0] = g_marks;
  out[1] = g_steps;
  out[2] = g_launched * g_graph_steps;
  out[3] = g_launched;
}

hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* st) {
  *st = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}

hipError_t __real_hipMalloc(void** p, size_t n);
hipError_t __wrap_hipMalloc(void** p, size_t n) {
  if (n > g_malloc_limit) return hipErrorOutOfMemory;
  ++g_mallocs;
  return __real_hipMalloc(p, n);
}
hipError_t __real_hipFree(void* p);
hipError_t __wrap_hipFree(void* p) {
  ++g_frees;
  return __real_hipFree(p);
}
hipError_t __real_hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode m);
hipError_t __wrap_hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode m) {
  g_own = true;
  return __real_hipStreamBeginCapture(s, m);
}
hipError_t __real_hipStreamEndCapture(hipStream_t s, hipGraph_t* g);
hipError_t __wrap_hipStreamEndCapture(hipStream_t s, hipGraph_t* g) {
  g_own = false;
  return __real_hipStreamEndCapture(s, g);
}
hipError_t __real_hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t g, hipGraphNode_t* n, char* l, size_t b);
hipError_t __wrap_hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t g, hipGraphNode_t* n, char* l, size_t b) {
  return g_fail_instantiate ? hipErrorOutOfMemory : __real_hipGraphInstantiate(x, g, n, l, b);
}
hipError_t __real_hipGraphLaunch(hipGraphExec_t x, hipStream_t s);
hipError_t __wrap_hipGraphLaunch(hipGraphExec_t x, hipStream_t s) {
  if (g_fail_launch == 0) return hipErrorOutOfMemory;
  if (g_fail_launch > 0) --g_fail_launch;
  ++g_launched;
  return __real_hipGraphLaunch(x, s);
}

// lbmib::launch_bead_stats(Dev const&, int, hipStream_t)
void __wrap__ZN5lbmib17launch_bead_statsERKNS_3DevEiP12ihipStream_t(const Dev&, int, hipStream_t) { ++g_marks; }
// lbmib::launch_interp_advance(Dev const&, hipStream_t): the closing launch of
// d.tick steps
void __wrap__ZN5lbmib21launch_interp_advanceERKNS_3DevEP12ihipStream_t(const Dev& d, hipStream_t) {
  if (g_own)
    g_graph_steps = d.tick;
  else
    g_steps += d.tick;
}
}
