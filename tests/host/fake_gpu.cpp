// A device for the host side of the C ABI (sim_api.cpp) on the CPU: the HIP calls it
// makes, with a memory of settable size and with captured graphs, and launchers that
// stand for the kernels by one number each. A state's first entry is its number (the
// start's plus the step), and so is the first entry of whatever is formed from it, so a
// solve can see whether the factor or the coarse operator it is given belongs to its matrix.

#include <hip/hip_runtime.h>
#include <sys/mman.h>

#include <algorithm>
#include <cstring>
#include <functional>
#include <map>
#include <vector>

#include "direct_kernels.h"
#include "kernels.h"

using namespace phisft;

namespace {

typedef std::vector<std::function<void()>> Work;

struct Capture {
  Work work;
  unsigned long long id;
};

struct {
  size_t total = size_t(1) << 34, used = 0;
  std::map<void*, size_t> live;
  std::map<hipStream_t, Capture> captures;
  unsigned long long ids = 0;
  int counts[8] = {};
  int iterations = 1000;   // of a solve, at most its cap
  int fail_in = 0;   // > 0: the allocation that fails, counted from now
} dev;

enum Count { kMallocs, kFactorised, kPasses, kStaleFactors, kCoarse, kIterated, kStaleCoarse };

void enqueue(hipStream_t st, std::function<void()> f) {
  auto c = dev.captures.find(st);
  if (c != dev.captures.end()) c->second.work.push_back(std::move(f));
  else f();
}

}  // namespace

extern "C" {

// what the tests set and read
void fake_memory(size_t bytes) { dev.total = bytes; }
void fake_iterations(int n) { dev.iterations = n; }
void fake_fail(int nth) { dev.fail_in = nth; }
size_t fake_used() { return dev.used; }
void fake_counts(int* out, int clear) {
  for (int k = 0; k < 8; ++k) out[k] = dev.counts[k];
  if (clear)
    for (int& c : dev.counts) c = 0;
}

hipError_t hipMalloc(void** p, size_t n) {
  ++dev.counts[kMallocs];
  if (dev.fail_in > 0 && --dev.fail_in == 0) return hipErrorOutOfMemory;
  if (n > dev.total - dev.used) return hipErrorOutOfMemory;
  void* q = mmap(nullptr, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  if (q == MAP_FAILED) return hipErrorOutOfMemory;
  dev.live[q] = n;
  dev.used += n;
  *p = q;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  auto i = dev.live.find(p);
  if (i == dev.live.end()) return p ? hipErrorInvalidValue : hipSuccess;
  munmap(p, i->second);
  dev.used -= i->second;
  dev.live.erase(i);
  return hipSuccess;
}
hipError_t hipMemGetInfo(size_t* fre, size_t* total) {
  *fre = dev.total - dev.used;
  *total = dev.total;
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemset(void* d, int v, size_t n) {
  memset(d, v, n);
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = nullptr; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.0f; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = reinterpret_cast<hipStream_t>(new int);
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
  delete reinterpret_cast<int*>(s);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) {
  dev.captures[s].id = ++dev.ids;
  return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t* g) {
  *g = reinterpret_cast<hipGraph_t>(new Work(std::move(dev.captures[s].work)));
  dev.captures.erase(s);
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st) {
  *st = dev.captures.count(s) ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamGetCaptureInfo(hipStream_t s, hipStreamCaptureStatus* st, unsigned long long* id) {
  hipStreamIsCapturing(s, st);
  if (*st == hipStreamCaptureStatusActive) *id = dev.captures[s].id;
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t g, hipGraphNode_t*, char*, size_t) {
  *e = reinterpret_cast<hipGraphExec_t>(new Work(*reinterpret_cast<Work*>(g)));
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t s) {
  for (auto& f : *reinterpret_cast<Work*>(e)) enqueue(s, f);
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) {
  delete reinterpret_cast<Work*>(g);
  return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t e) {
  delete reinterpret_cast<Work*>(e);
  return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode*) { return hipSuccess; }

}  // extern "C"

namespace phisft {

void launch_fill_int(int*, int, int, hipStream_t) {}
void launch_fill_double(double* p, long n, double v, hipStream_t st) {
  if (n > 0) enqueue(st, [=] { p[0] = v; });
}
void launch_elements(const Mesh&, const Elem& el, const double* x, const double*, const double*,
                     const double*, double, int*, hipStream_t st) {
  double* f = el.tri_f;
  enqueue(st, [=] { f[0] = x[0]; });
}
template <typename T, typename TM>
void launch_assemble(const Mesh&, const Elem& el, const AssembleArgs<T, TM>& a, hipStream_t st) {
  const double* f = el.tri_f;
  enqueue(st, [=] { a.A[0] = (TM)f[0]; });
}
template <typename TM>
size_t pcg_lds_bytes(int, int, int, int, int, int) { return 1024; }
template <typename TM>
hipError_t pcg_prepare(size_t, int, int, bool, int) { return hipSuccess; }
template <typename TM>
hipError_t pcg_occupancy(int, size_t, int, int, bool, int, bool, int* n) { *n = 1; return hipSuccess; }
template <typename TM>
void launch_pcg(const Mesh& m, const SolverPlan&, const SolverWork&, const Coarse& cs,
                const PcgArgs<TM>& a, hipStream_t st, bool) {
  enqueue(st, [=] {
    if (a.left && *a.left == 0) return;
    ++dev.counts[kIterated];
    if (cs.nagg && cs.xinv[0] != (float)a.A[0]) ++dev.counts[kStaleCoarse];
    a.sol[0] = a.A[0];
    for (int b = 0; a.iters && b < m.ninst; ++b) a.iters[b] = std::min(dev.iterations, a.max_iter);
  });
}
template <typename TM>
bool launch_coarse_setup(const Mesh& m, const SolverWork&, const Coarse& c, const double*, const TM* A,
                         long long, const std::vector<int>&, hipStream_t st) {
  if (c.nagg == 0) return false;
  enqueue(st, [=] {
    if (c.left && *c.left == 0) return;
    ++dev.counts[kCoarse];
    c.xinv[0] = (float)A[0];
  });
  return true;
}
hipError_t gj_sweep_occupancy(int, int* n) { *n = 2; return hipSuccess; }
template <typename T>
void launch_update(const Mesh&, const double* xp, const double*, const double*, double, double* xn,
                   double*, T*, int*, hipStream_t st) {
  enqueue(st, [=] { xn[0] = xp[0] + 1.0; });
}
template <typename T>
void launch_init_state(const Mesh&, const T* x0, const T*, double* xs, double*, int*, hipStream_t st) {
  enqueue(st, [=] { xs[0] = x0[0]; });
}
template <typename T>
void launch_adj_pre(const Mesh&, const T*, double, double*, const double*, double*, int*, hipStream_t) {}
template <typename T>
void launch_adj_elements(const Mesh&, const Elem&, const AdjArgs<T>&, hipStream_t) {}
template <typename T>
void launch_adj_rows(const Mesh&, const Elem&, const AdjArgs<T>&, hipStream_t) {}
template <typename T>
void launch_adj_final(const Mesh&, const double*, const double*, T*, T*, hipStream_t) {}
void launch_material_sum(const Mesh&, const Elem&, double*, double*, hipStream_t) {}
template <typename T>
void launch_frame_loss(const T*, const T*, int, const int*, const int*, int, int, double*, T*,
                       hipStream_t) {}
hipError_t noalloc_scratch(void** out) {
  static char scratch[kNoAllocScratchBytes];
  *out = scratch;
  return hipSuccess;
}

hipError_t ds_prepare(int* n) { *n = 2; return hipSuccess; }
void launch_ds_run(const DsArgs* args, double* fac, const DsTask*, int, bool factor, int,
                   const int* left, hipStream_t st) {
  enqueue(st, [=] {
    if (left && *left == 0) return;
    if (!left) args->left[0] = args->left[1] = 0;
    ++dev.counts[factor ? kFactorised : kPasses];
    if (factor) fac[0] = args->A[0];
    else if (fac[0] != args->A[0]) ++dev.counts[kStaleFactors];
    args->sol[0] = fac[0];
  });
}
void launch_ds_add(const DsArgs&, const DsAccept&, const double*, const int*, hipStream_t) {}
void launch_ds_resid(const DsArgs& a, const DsAccept& o, const DsRows* tasks, int n, hipStream_t st) {
  enqueue(st, [=] {
    for (int k = 0; k < n; ++k) {
      const int b = tasks[k].sheet;
      if (o.again && o.done[b]) continue;
      o.done[b] = a.sol[0] == a.A[0] && o.tol > 0.0;
      if (!o.done[b] && (k == 0 || tasks[k - 1].sheet != b)) ++*o.left;
      if (o.iters && o.done[b]) o.iters[b] = 1;
    }
  });
}

#define INSTANTIATE(T)                                                                             \
  template void launch_assemble<T, double>(const Mesh&, const Elem&,                              \
                                           const AssembleArgs<T, double>&, hipStream_t);          \
  template void launch_assemble<T, float>(const Mesh&, const Elem&, const AssembleArgs<T, float>&, \
                                          hipStream_t);                                            \
  template size_t pcg_lds_bytes<T>(int, int, int, int, int, int);                                  \
  template hipError_t pcg_prepare<T>(size_t, int, int, bool, int);                                 \
  template hipError_t pcg_occupancy<T>(int, size_t, int, int, bool, int, bool, int*);              \
  template void launch_pcg<T>(const Mesh&, const SolverPlan&, const SolverWork&, const Coarse&,    \
                              const PcgArgs<T>&, hipStream_t, bool);                               \
  template bool launch_coarse_setup<T>(const Mesh&, const SolverWork&, const Coarse&,              \
                                       const double*, const T*, long long,                         \
                                       const std::vector<int>&, hipStream_t);                      \
  template void launch_update<T>(const Mesh&, const double*, const double*, const double*, double, \
                                 double*, double*, T*, int*, hipStream_t);                         \
  template void launch_init_state<T>(const Mesh&, const T*, const T*, double*, double*, int*,      \
                                     hipStream_t);                                                 \
  template void launch_adj_pre<T>(const Mesh&, const T*, double, double*, const double*, double*,  \
                                  int*, hipStream_t);                                              \
  template void launch_adj_elements<T>(const Mesh&, const Elem&, const AdjArgs<T>&, hipStream_t);  \
  template void launch_adj_rows<T>(const Mesh&, const Elem&, const AdjArgs<T>&, hipStream_t);      \
  template void launch_adj_final<T>(const Mesh&, const double*, const double*, T*, T*,             \
                                    hipStream_t);                                                  \
  template void launch_frame_loss<T>(const T*, const T*, int, const int*, const int*, int, int,    \
                                     double*, T*, hipStream_t);
INSTANTIATE(double)
INSTANTIATE(float)

}  // namespace phisft
