// A HIP runtime without a device, loaded ahead of libmgmi.so to test the host side of a
// solve on the CPU.  Device memory is host memory, kernels do nothing, and every stream is
// one queue in which only the kernels of the stopping rule act: the start of a solve clears
// its count of checks, and each check reports to the solve's pinned state as the real one
// does, the check number fake_stop_at's value (as the solve starts) with the done flag.  hipStreamQuery runs one entry of the
// queue, a synchronization all of them, so the host meets every check as late as it can.
#include <hip/hip_runtime_api.h>

#include <cstdlib>
#include <cstring>
#include <deque>
#include <map>
#include <string>
#include <vector>

namespace {

enum Kind { kNone, kStart, kCheck };
struct Entry {
  Kind kind;
  int *report;  // {done, checks} (mg) or {checks, done} (red-black coarsening)
  bool rbc;
  int stop_at;  // of a start: the check that stops its solve
};

std::map<const void *, std::string> g_names;
std::deque<Entry> g_queue;
std::vector<Entry> *g_capture = nullptr;
std::vector<std::vector<Entry> *> g_graphs;
int g_checks = 0, g_stop = 0, g_stop_at = 1 << 30;
int g_kernels = 0, g_graph_launches = 0, g_fail_in = 0;
hipError_t g_error = hipSuccess;
dim3 g_grid, g_block;

void run_one() {
  const Entry e = g_queue.front();
  g_queue.pop_front();
  if (e.kind == kStart) {
    g_checks = 0;
    g_stop = e.stop_at;
  }
  if (e.kind != kCheck || g_checks >= g_stop) return;
  ++g_checks;
  e.report[e.rbc ? 1 : 0] = g_checks >= g_stop;
  e.report[e.rbc ? 0 : 1] = g_checks;
  if (!e.rbc) e.report[2] = g_checks >= g_stop ? 1 : 0;  // status
}
void drain() {
  while (!g_queue.empty()) run_one();
}
// The launch that was asked to fail.
bool refused() { return g_fail_in > 0 && --g_fail_in == 0; }

}  // namespace

extern "C" {

void fake_stop_at(int check) { g_stop_at = check; }
void fake_fail_launch(int nth) { g_fail_in = nth; }
void fake_counts(int *kernels, int *graphs) {
  *kernels = g_kernels;
  *graphs = g_graph_launches;
  g_kernels = g_graph_launches = 0;
}

void **__hipRegisterFatBinary(const void *) {
  static void *mod;
  return &mod;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *fn, char *, const char *name, unsigned, void *, void *, dim3 *, dim3 *,
                           int *) {
  g_names[fn] = name;
}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t, hipStream_t) {
  g_grid = g;
  g_block = b;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *m, hipStream_t *s) {
  *g = g_grid;
  *b = g_block;
  *m = 0;
  *s = nullptr;
  return hipSuccess;
}

hipError_t hipLaunchKernel(const void *fn, dim3, dim3, void **args, size_t, hipStream_t) {
  if (!g_capture) {
    ++g_kernels;
    if (refused()) return g_error = hipErrorLaunchFailure;
  }
  const std::string &name = g_names[fn];
  Entry e{kNone, nullptr, false, g_stop_at};
  if (name.find("k_state_init") != std::string::npos || name.find("k_rbc_start") != std::string::npos) {
    e.kind = kStart;
  } else if (name.find("k_rbc_check") != std::string::npos) {
    e = {kCheck, *(int **)args[1], true, 0};
  } else if (name.find("k_check") != std::string::npos && *(int *)args[3] != 0) {
    e = {kCheck, *(int **)args[4], false, 0};
  }
  if (e.kind == kCheck && e.report == nullptr) e.kind = kNone;
  if (g_capture)
    g_capture->push_back(e);
  else
    g_queue.push_back(e);
  return hipSuccess;
}
hipError_t hipGetLastError() {
  const hipError_t e = g_error;
  g_error = hipSuccess;
  return e;
}
const char *hipGetErrorString(hipError_t) { return "fake error"; }

hipError_t hipStreamQuery(hipStream_t) {
  if (g_queue.empty()) return hipSuccess;
  run_one();
  return hipErrorNotReady;
}
hipError_t hipStreamSynchronize(hipStream_t) {
  drain();
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return hipStreamSynchronize(nullptr); }
hipError_t hipEventQuery(hipEvent_t) { return hipStreamSynchronize(nullptr); }

hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) {
  g_graphs.push_back(new std::vector<Entry>);
  g_capture = g_graphs.back();
  return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) {
  *g = (hipGraph_t)g_capture;
  g_capture = nullptr;
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t g, hipGraphNode_t *, char *, size_t) {
  *x = (hipGraphExec_t)g;
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t) {
  ++g_graph_launches;
  if (refused()) return hipErrorLaunchFailure;
  for (const Entry &e : *(std::vector<Entry> *)x) g_queue.push_back(e);
  return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }

hipError_t hipMalloc(void **p, size_t n) { return (*p = calloc(1, n)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void *p) {
  drain();  // as the real one does
  free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipHostFree(void *p) { return hipFree(p); }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
  memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
  return hipMemcpy(d, s, n, hipMemcpyDefault);
}
hipError_t hipMemsetAsync(void *, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipGetDevice(int *d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int) {
  *v = a == hipDeviceAttributeMaxSharedMemoryPerBlock ? 160 * 1024 : 256;
  return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) {
  *n = 2;
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
  *s = (hipStream_t)0x1;
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
  *e = (hipEvent_t)0x1;
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }

}  // extern "C"
