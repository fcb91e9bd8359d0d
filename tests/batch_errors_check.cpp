// Host check of dfw_batch_run's error exits: the library's host code linked against the runtime below, in
// which "device" memory is host memory, kernels do nothing and one chosen call fails.  With a final time and
// more steps than a chunk the run is several launches with host waits between; whichever of them fails, the
// call has to return the error with nothing left running on the caller's buffers, keep no half-made state for
// the next call, and the plan has to give back everything it took.  Prints one line per fault: name, the
// number of violations.  Built and run by tests/test_batch_errors.py.
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "../include/dfweno.h"

namespace {
std::string g_fail_name;  // the call that fails ...
int g_fail_at = 0;        // ... and which one of them, from 1; 0: none
int g_seen = 0;
bool g_pending = false, g_capturing = false;
int g_events = 0, g_pinned = 0, g_graphs = 0, g_execs = 0, g_replays = 0;

bool fails(const char* name) { return g_fail_at && g_fail_name == name && ++g_seen == g_fail_at; }
template <class T>
T handle() {
  static char pool[1 << 16];
  static size_t used = 0;
  return reinterpret_cast<T>(&pool[++used % sizeof(pool)]);
}
}  // namespace

extern "C" {
void** __hipRegisterFatBinary(const void*) { return handle<void**>(); }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3*, dim3*, size_t*, hipStream_t*) { return hipSuccess; }
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) {
  if (!g_capturing) g_pending = true;
  return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "injected"; }
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { return *v = 256, hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) { return *p = nullptr, hipErrorInvalidSymbol; }
hipError_t hipMalloc(void** p, size_t n) { return *p = std::calloc(1, n), hipSuccess; }
hipError_t hipFree(void* p) { return std::free(p), hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  if (fails("hipHostMalloc")) return hipErrorOutOfMemory;
  ++g_pinned;
  *p = std::malloc(n);
  std::memset(*p, 1, n);  // no kernel runs to clear it: grids are always left to advance
  return hipSuccess;
}
hipError_t hipHostFree(void* p) { return --g_pinned, std::free(p), hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { return std::memcpy(d, s, n), hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  if (fails("hipMemcpyAsync")) return hipErrorUnknown;
  return g_pending = true, std::memcpy(d, s, n), hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { return *s = handle<hipStream_t>(), hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return g_pending = false, hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return g_capturing = true, hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
  g_capturing = false;
  if (fails("hipStreamEndCapture")) return *g = nullptr, hipErrorUnknown;
  return ++g_graphs, *g = handle<hipGraph_t>(), hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  if (fails("hipGraphInstantiate")) return hipErrorOutOfMemory;
  return ++g_execs, *e = handle<hipGraphExec_t>(), hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) {
  if (fails("hipGraphLaunch")) return hipErrorLaunchFailure;
  return ++g_replays, g_pending = true, hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return --g_graphs, hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return --g_execs, hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  if (fails("hipEventCreateWithFlags")) return hipErrorOutOfMemory;
  return ++g_events, *e = handle<hipEvent_t>(), hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t) { return --g_events, hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { return *ms = 0, hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return fails("hipEventRecord") ? hipErrorUnknown : hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) {
  return fails("hipEventSynchronize") ? hipErrorUnknown : hipSuccess;  // of the chunk before the one in flight
}
}

int main() {
  constexpr int kSteps = 70, kChunks = 5;  // chunks of 16 steps
  const dfw_grid grid = {12, 10, 0.1, 0.1, DFW_BC_PERIODIC, DFW_BC_PERIODIC};
  dfw_params p{};
  p.gamma = 1.4, p.cfl = 0.5, p.alpha_thres = 0.5, p.d_h = p.d_l = 0.85, p.eps_weno = 1e-6, p.c1 = 0.01, p.c2 = 5.0;
  p.t_end = 1.0;
  struct Fault {
    const char* name;
    int calls;  // the first so many of them in turn
    bool graph, direct;
  };
  const Fault faults[] = {{"none", 1, true, true},
                          {"hipEventCreateWithFlags", 2, true, true},
                          {"hipHostMalloc", 1, true, true},
                          {"hipStreamEndCapture", kChunks, true, false},
                          {"hipGraphInstantiate", kChunks, true, false},
                          {"hipGraphLaunch", kChunks, true, false},
                          {"hipEventRecord", kChunks, true, true},
                          {"hipEventSynchronize", kChunks - 2, true, true},
                          {"hipMemcpyAsync", 1, true, true}};
  for (const Fault& f : faults)
    for (int graph = 0; graph < 2; ++graph) {
      if (!(graph ? f.graph : f.direct)) continue;
      int bad = 0;
      for (int at = 1; at <= f.calls; ++at) {
        const int events = g_events, pinned = g_pinned, graphs = g_graphs, execs = g_execs;
        dfw_batch* b = nullptr;
        size_t nw = 0, na = 0, nws = 0;
        bad += dfw_batch_plan(&grid, 1, &p, DFW_F64, 0, &b) != DFW_OK;
        bad += dfw_batch_layout(b, nullptr, nullptr, &nw, &na, &nws) != DFW_OK;
        std::vector<double> W(nw), A(na);
        void* ws = std::aligned_alloc(256, (nws + 255) / 256 * 256);
        std::memset(ws, 0, nws);
        const bool none = std::strcmp(f.name, "none") == 0;
        g_fail_name = f.name, g_fail_at = none ? 0 : at, g_seen = 0, g_pending = false;
        double t = 0;
        int32_t fail = 0;
        auto run = [&] {
          return dfw_batch_run(b, W.data(), A.data(), kSteps, ws, nws, graph, nullptr, &t, &fail, nullptr);
        };
        // no kernel runs, so the control block still names a failure at step 0: that status is a full run's
        const dfw_status s = run();
        bad += s != (none ? DFW_ENONPHYS : DFW_EHIP);
        bad += !none && g_seen != at;  // the fault was met
        bad += g_pending;              // work left on the caller's buffers
        g_fail_at = 0, g_replays = 0;
        bad += run() != DFW_ENONPHYS;
        bad += g_replays != (graph ? kChunks : 0) || g_pending;
        dfw_batch_free(b);
        bad += g_events != events || g_pinned != pinned || g_graphs != graphs || g_execs != execs;
        std::free(ws);
      }
      std::printf("%s_%s %d\n", f.name, graph ? "graph" : "direct", bad);
    }
  return 0;
}
