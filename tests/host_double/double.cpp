// A stand-in for the GPU under the library's host sources, for tests of the
// host logic (server scheduling, failures, host copies) on the CPU.
//
// Device memory is host memory and work runs when it is enqueued, or when its
// graph is launched.  A domain's state is a count of the steps it has taken:
// launch_init writes 0 into the current buffer of the CH group, one step
// reads the current buffer and writes the count plus one into the other, and
// launch_macro returns the count in c.  Any call can be made to fail, as the
// n-th one of its name from now.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <functional>
#include <map>
#include <mutex>
#include <set>
#include <string>
#include <thread>
#include <vector>

#include "host_internal.h"

struct ihipGraph {
  std::vector<std::function<void()>> ops;
};
struct ihipStream {
  bool pending = false;
  std::set<ihipStream *> joined;   // streams whose work this one waits for
  ihipGraph *capture = nullptr;    // the graph its work is recorded into
};
struct ihipEvent {
  std::set<ihipStream *> src;
  ihipGraph *capture = nullptr;
};

namespace {

std::recursive_mutex g_mu;
std::map<std::string, int> g_fail;        // calls until that one fails
std::map<std::string, int64_t> g_calls;
std::set<std::thread::id> g_threads;      // that made a runtime call
std::set<ihipStream *> g_streams;
thread_local hipError_t t_last = hipSuccess;
ihipStream g_null;
int64_t g_live_host = 0, g_unsafe = 0;
size_t g_strips = 0;                      // blocks of the largest launch

struct Launch {
  int N, precision, ty, domains, graph;
  ihipStream *st;
};
std::vector<Launch> g_launches;

// counts the call and says whether it fails
hipError_t enter(const char *name) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  g_threads.insert(std::this_thread::get_id());
  ++g_calls[name];
  auto it = g_fail.find(name);
  if (it == g_fail.end() || --it->second > 0) return hipSuccess;
  g_fail.erase(it);
  t_last = std::strcmp(name, "hipHostMalloc") == 0 ? hipErrorOutOfMemory : hipErrorLaunchFailure;
  return t_last;
}
#define ENTER(name)                                             \
  std::lock_guard<std::recursive_mutex> lk(g_mu);               \
  if (hipError_t e_ = enter(name)) return e_

ihipStream *str(hipStream_t st) { return st ? st : &g_null; }

void work(hipStream_t st, std::function<void()> f) {
  ihipStream *s = str(st);
  if (s->capture) {
    s->capture->ops.push_back(std::move(f));
  } else {
    s->pending = true;
    f();
  }
}
// what the kernel launchers return
hipError_t launched() {
  const hipError_t e = t_last;
  t_last = hipSuccess;
  return e;
}

}  // namespace

const char *hipGetErrorString(hipError_t e) { return e ? "error of the double" : "no error"; }
hipError_t hipGetLastError() { return launched(); }
hipError_t hipGetDevice(int *dev) {
  ENTER("hipGetDevice");
  *dev = 0;
  return hipSuccess;
}
hipError_t hipSetDevice(int) {
  ENTER("hipSetDevice");
  return hipSuccess;
}
hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int) {
  p->multiProcessorCount = nplbm::kComputeUnits;
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() {
  for (ihipStream *s : g_streams) s->pending = false;
  g_null.pending = false;
  return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t bytes) {
  ENTER("hipMalloc");
  *p = aligned_alloc(256, (bytes + 255) & ~(size_t)255);
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void *p) {
  ENTER("hipFree");
  for (ihipStream *s : g_streams) g_unsafe += p && s->pending;
  free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t bytes, unsigned) {
  ENTER("hipHostMalloc");
  *p = malloc(bytes);
  ++g_live_host;
  return hipSuccess;
}
hipError_t hipHostFree(void *p) {
  ENTER("hipHostFree");
  free(p);
  --g_live_host;
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void *dst, const void *src, size_t bytes, hipMemcpyKind, hipStream_t st) {
  ENTER("hipMemcpyAsync");
  work(st, [=] { std::memcpy(dst, src, bytes); });
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *st, unsigned) {
  ENTER("hipStreamCreateWithFlags");
  *st = new ihipStream;
  g_streams.insert(*st);
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t st) {
  ENTER("hipStreamDestroy");
  g_unsafe += st->pending;
  g_streams.erase(st);
  delete st;
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t st) {
  ENTER("hipStreamSynchronize");
  ihipStream *s = str(st);
  for (ihipStream *j : s->joined)
    if (g_streams.count(j)) j->pending = false;
  s->joined.clear();
  s->pending = false;
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t st, hipEvent_t ev, unsigned) {
  ENTER("hipStreamWaitEvent");
  ihipStream *s = str(st);
  s->joined.insert(ev->src.begin(), ev->src.end());
  if (ev->capture) s->capture = ev->capture;
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *ev, unsigned) {
  ENTER("hipEventCreateWithFlags");
  *ev = new ihipEvent;
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t ev) {
  ENTER("hipEventDestroy");
  delete ev;
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t ev, hipStream_t st) {
  ENTER("hipEventRecord");
  ihipStream *s = str(st);
  ev->src = s->joined;
  ev->src.insert(s);
  ev->capture = s->capture;
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) {
  ENTER("hipEventSynchronize");
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t st, hipStreamCaptureMode) {
  ENTER("hipStreamBeginCapture");
  st->capture = new ihipGraph;
  return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t st, hipGraph_t *g) {
  ENTER("hipStreamEndCapture");
  *g = st->capture;
  for (ihipStream *s : g_streams)
    if (s->capture == *g) {
      s->capture = nullptr;
      s->joined.clear();
    }
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t g, void *, char *, size_t) {
  ENTER("hipGraphInstantiate");
  *x = new ihipGraph(*g);
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t st) {
  ENTER("hipGraphLaunch");
  const size_t before = g_launches.size();
  work(st, [=] {
    for (auto &f : x->ops) f();
  });
  for (size_t i = before; i < g_launches.size(); ++i) g_launches[i].graph = 1;
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) {
  delete g;
  return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t x) {
  delete x;
  return hipSuccess;
}

namespace nplbm {

namespace {

void advance(const DomDesc &D, int substep) {
  if (substep >= D.steps_left) return;
  const int par = (substep + D.parity0) & 1;
  int64_t n;
  std::memcpy(&n, D.h[par], sizeof n);
  ++n;
  std::memcpy(D.h[par ^ 1], &n, sizeof n);
}

}  // namespace

hipError_t launch_geom_step(int N, int precision, int scheme, const StepGeom &g, const StepArgs &a,
                            int nblocks, const DomDesc *one, hipStream_t st) {
  ENTER("launch_geom_step");
  const DomDesc desc = one ? *one : DomDesc();
  const bool single = one != nullptr;
  const int ty = g.ty;
  work(st, [=] {
    int domains = 0;
    if (single) {
      advance(desc, a.substep);
      domains = 1;
    } else {
      for (int b = 0; b < nblocks; ++b) {
        const StripDesc &s = a.strips[b];
        if (s.dom < 0 || s.x0 || s.y0) continue;
        advance(a.doms[s.dom], a.substep);
        ++domains;
      }
    }
    g_launches.push_back({N, precision, ty, domains, 0, str(st)});
  });
  return launched();
}
hipError_t launch_step3(int, int, int, const StepArgs &a, int, int, int, int, int, hipStream_t st) {
  ENTER("launch_step3");
  work(st, [=] { advance(*a.doms, a.substep); });
  return launched();
}
hipError_t launch_progress(DomDesc *descs, const Progress &p, hipStream_t st) {
  ENTER("launch_progress");
  work(st, [=] {
    for (int j = 0; j < kProgressSlots; ++j) {
      if (p.left[j] < 0) continue;
      descs[p.base + j].parity0 = (p.odd[j / 32] >> (j % 32)) & 1;
      descs[p.base + j].steps_left = p.left[j];
    }
  });
  return launched();
}
hipError_t launch_init(const DomDesc *, const DomDesc &dd, int, const double *, const double *,
                       const double *, const double *, const double *, double *, double *,
                       hipStream_t st) {
  ENTER("launch_init");
  void *h = dd.h[dd.parity0];
  work(st, [=] { std::memset(h, 0, sizeof(int64_t)); });
  return launched();
}
hipError_t launch_init3(const DomDesc *d, const DomDesc &dd, int p, const double *a,
                        const double *b, const double *c, const double *e, const double *f,
                        double *g, double *h, hipStream_t st) {
  return launch_init(d, dd, p, a, b, c, e, f, g, h, st);
}
hipError_t launch_macro(const DomDesc *, const DomDesc &dd, int, int parity, double *, double *,
                        double *, double *c, double *, double *, double *, hipStream_t st) {
  ENTER("launch_macro");
  const void *h = dd.h[parity];
  const size_t n = (size_t)dd.nx * dd.ny * dd.nz * dd.N;
  work(st, [=] {
    int64_t k;
    std::memcpy(&k, h, sizeof k);
    std::fill(c, c + n, (double)k);
  });
  return launched();
}
hipError_t launch_macro3(const DomDesc *d, const DomDesc &dd, int p, int par, double *a, double *b,
                         double *e, double *c, double *f, double *g, hipStream_t st) {
  return launch_macro(d, dd, p, par, a, b, e, c, f, g, nullptr, st);
}
hipError_t launch_diag(const DomDesc *, const DomDesc &, int, int, double *, int, double *,
                       hipStream_t) {
  return launched();
}
hipError_t launch_diag3(const DomDesc *, const DomDesc &, int, int, double *, int, double *,
                        hipStream_t) {
  return launched();
}
hipError_t launch_laplace(const double *, int, int, int, double, double, double, double, double,
                          double *, int, double *, hipStream_t) {
  return launched();
}
hipError_t launch_copy(void *, const void *, size_t, hipStream_t) { return launched(); }
hipError_t static_diag_scratch(double **out) {
  static double s[kStaticDiagDoubles];
  *out = s;
  return hipSuccess;
}
int diag_blocks(int64_t n) { return (int)std::min<int64_t>((n + 255) / 256, 1024); }
int step_blocks_per_cu(int, int, int, int) { return 1; }
int step3_blocks_per_cu(int, int, int) { return 1; }
int step_max_bw(int, int, int) { return 256; }
int step3_ty(int, int, int, int, int) { return 4; }
int step3_march_ty(int, int) { return 4; }

}  // namespace nplbm

extern "C" {

// the n-th call named so from now fails
void double_fail(const char *name, int n) { g_fail[name] = n; }
int64_t double_calls(const char *name) { return g_calls[name]; }
void double_reset() {
  g_fail.clear();
  g_calls.clear();
  g_threads.clear();
  g_launches.clear();
  g_unsafe = 0;
  t_last = hipSuccess;
  (void)hipDeviceSynchronize();
}
void *double_stream() {
  hipStream_t st;
  (void)hipStreamCreateWithFlags(&st, 0);
  return st;
}
int double_threads() { return (int)g_threads.size(); }
// memory freed or streams destroyed while a stream had work that nothing waited for
int64_t double_unsafe() { return g_unsafe; }
int64_t double_pinned() { return g_live_host; }
// whether the plan of a 3-D domain has room for the node kernels' array of C
int double_node_array(const nplbm_params *p) { return nplbm::plan_layout(p).c3 != 0; }
int double_launches() { return (int)g_launches.size(); }
// launch i: N, precision, tile rows (0: strips), domains, from a graph, stream
void double_launch(int i, int64_t *out) {
  const Launch &l = g_launches[i];
  const int64_t v[6] = {l.N, l.precision, l.ty, l.domains, l.graph, (int64_t)l.st};
  std::memcpy(out, v, sizeof v);
}
}
