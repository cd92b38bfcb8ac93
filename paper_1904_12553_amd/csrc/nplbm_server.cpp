// nplbm_server.cpp -- continuous batching of many small domains on one GPU
// (the serving part of the C ABI in include/nplbm.h).
//
// Every resident domain keeps its distributions in its own device
// allocation for its whole life.  One pump = admit what fits, then one
// quantum of Q steps in which every resident domain of a given (N,
// precision, scheme, kernel) group is advanced by the same step kernel launch,
// driven by a packed strip table over all the group's domains.  Groups that
// fit the Infinity Cache together run side by side, one such set after the
// other, and last those of the domains beyond it.  The
// launches of a quantum are captured into a HIP graph and replayed once a
// resident set outlasts its first quantum; per-domain progress (which
// ping-pong buffer is current, how many of the Q sub-steps it still needs) is
// written into the device descriptors before each quantum, so a domain that
// finishes mid-quantum simply stops.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <climits>
#include <cmath>
#include <cstring>
#include <deque>
#include <map>
#include <memory>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "host_internal.h"
#include "nplbm.h"
#include "nplbm_internal.h"

using namespace nplbm;

namespace {

// side streams of the quantum graph (groups beyond this share them)
constexpr int kSideStreams = 4;

double now_s() {
  using namespace std::chrono;
  return duration<double>(steady_clock::now().time_since_epoch()).count();
}

struct Req {
  uint64_t ticket = 0;
  nplbm_params p{};
  std::vector<double> sigma, rho, mu, mob, tau;
  std::vector<double> c, u;
  bool has_u = false;
  int64_t nsteps = 0;
  int64_t done_steps = 0;
  // 0 queued, 1 resident, 2 done, 3 failed; written and read only under the
  // server's mutex, after everything it publishes (results, times) is written
  int state = 0;
  int err = 0;      // failed request: the error code and message
  std::string msg;
  double t_submit = 0, t_admit = 0, t_done = 0;
  // resident
  Derived d;
  Layout L;
  size_t bytes = 0;
  unsigned char *base = nullptr;
  int slot = -1;
  DomDesc desc{};
  // results: the device planes c, u and p as they lie, from L.c on (not
  // cleared first)
  std::unique_ptr<double[]> out;
};

}  // namespace

struct nplbm_server {
  size_t budget = 0, used = 0;
  int max_slots = 0, quantum = 1;
  hipStream_t stream = nullptr;
  std::mutex mu;
  uint64_t next_ticket = 1;
  std::deque<Req *> queue;
  std::map<uint64_t, Req *> reqs;
  std::vector<Req *> slots;  // resident requests by slot (nullptr = free)
  DomDesc *descs_dev = nullptr;
  StripDesc *strips_dev = nullptr;
  size_t strips_cap = 0;
  struct Group {
    int N, precision, scheme;
    StepGeom geom;
    size_t off, count;
    int64_t bytes;  // both copies of the states of its domains
    int wave;       // groups of one wave run side by side, waves in turn
  };
  std::vector<Group> groups;
  int waves = 0;
  // side streams and events of a quantum: each group's chain of launches
  // runs on its own stream, so the groups of a wave run side by side
  std::vector<hipStream_t> side;
  hipEvent_t fork = nullptr;
  std::vector<hipEvent_t> join;
  hipGraphExec_t graph = nullptr;  // a quantum of the resident set, once that set has lasted
  bool dirty = true;               // the resident set changed since the tables were built
  double node_updates = 0, busy = 0;
  int64_t completed = 0;
  // completion latencies (submit to done) of every finished request, and
  // the first submission / last completion times (under the mutex)
  std::vector<double> lat;
  double t_first = -1.0, t_last = 0.0;
  nplbm_server() { copy_users(1); }
  ~nplbm_server() { copy_users(-1); }
};

namespace {

void release(nplbm_server *s, Req *r) {
  if (r->base) (void)hipFree(r->base);
  r->base = nullptr;
  s->used -= r->bytes;
  if (r->slot >= 0) s->slots[r->slot] = nullptr;
  r->slot = -1;
}

int admit(nplbm_server *s, Req *r) {
  void *m = nullptr;
  hipError_t e = hipMalloc(&m, r->bytes);
  if (e != hipSuccess) {
    forget_hip_error();
    return fail(NPLBM_ENOMEM, "hipMalloc(%zu): %s", r->bytes, hipGetErrorString(e));
  }
  r->base = static_cast<unsigned char *>(m);
  s->used += r->bytes;
  int slot = -1;
  for (int i = 0; i < s->max_slots; ++i)
    if (!s->slots[i]) {
      slot = i;
      break;
    }
  r->slot = slot;
  s->slots[slot] = r;
  DomDesc &D = r->desc;
  std::memset(&D, 0, sizeof D);
  for (int b = 0; b < 2; ++b) {
    D.h[b] = r->base + r->L.h[b];
    D.g[b] = r->base + r->L.g[b];
  }
  D.prev[0] = r->base + r->L.prev[0];
  D.prev[1] = r->base + r->L.prev[1];
  for (int G = 0; G < 3; ++G) {
    D.ps[G] = r->L.ps[G];
    D.rs[G] = r->L.rs[G];
  }
  D.nx = r->p.nx;
  D.ny = r->p.ny;
  D.nz = 1;
  D.pitch = r->L.pitch;
  D.wall = r->p.wall_y;
  D.N = r->p.N;
  D.parity0 = 0;
  D.steps_left = INT_MAX;
  D.scheme = step_scheme(&r->p);
  D.cd = r->d.cd;
  D.cf = r->d.cf;
  const size_t n = (size_t)r->p.nx * r->p.ny;
  double *cdev = reinterpret_cast<double *>(r->base + r->L.c);
  double *udev = reinterpret_cast<double *>(r->base + r->L.u);
  e = hipMemcpyAsync(s->descs_dev + slot, &D, sizeof D, hipMemcpyHostToDevice, s->stream);
  if (e == hipSuccess)
    e = hipMemcpyAsync(cdev, r->c.data(), r->c.size() * 8, hipMemcpyHostToDevice, s->stream);
  if (e == hipSuccess && r->has_u)
    e = hipMemcpyAsync(udev, r->u.data(), 2 * n * 8, hipMemcpyHostToDevice, s->stream);
  if (e == hipSuccess)
    e = launch_init(s->descs_dev + slot, D, r->p.precision, r->d.P1, r->d.PN, r->d.P0, cdev,
                    r->has_u ? udev : nullptr,
                    reinterpret_cast<double *>(r->base + r->L.phi),
                    reinterpret_cast<double *>(r->base + r->L.C), s->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(s->stream);
  if (e != hipSuccess) {
    release(s, r);
    return hip_fail(e, "admission");
  }
  std::vector<double>().swap(r->c);
  std::vector<double>().swap(r->u);
  r->t_admit = now_s();
  r->done_steps = 0;
  s->dirty = true;
  return NPLBM_OK;
}

// Rebuild the packed strip tables (one per (N, precision, step-kernel
// scheme, kernel) group) and the order in which a quantum runs them.
int rebuild(nplbm_server *s) {
  if (s->graph) {
    (void)hipGraphExecDestroy(s->graph);
    s->graph = nullptr;
  }
  s->groups.clear();
  s->waves = 0;
  std::vector<StripDesc> all, g;
  for (int sch : {kSchemeCentral, kSchemeMixed, kSchemeRemark1})
    for (int prec : {32, 64})
      for (int N = 2; N <= kMaxN; ++N)
        // one table per kernel: strips (ty = 0) and tiles of each height
        // of domains whose own state fits the cache, in tables that fit it,
        // and of all those beyond it, which read HBM whatever runs beside them
        for (int ty : {0, 4, 8})
          for (bool fits : {true, false}) {
            StepGeom geom{};
            int64_t bytes = 0;
            auto close = [&]() {
              if (g.empty()) return;
              xcd_order(g);
              s->groups.push_back({N, prec, sch, geom, all.size(), g.size(), bytes, 0});
              all.insert(all.end(), g.begin(), g.end());
              g.clear();
              bytes = 0;
            };
            for (int slot = 0; slot < s->max_slots; ++slot) {
              Req *r = s->slots[slot];
              if (!r || r->p.N != N || r->p.precision != prec || step_scheme(&r->p) != sch)
                continue;
              const StepGeom rg = domain_geom(&r->p, true);
              const int64_t b = 2 * (int64_t)(r->L.gbytes[0] + r->L.gbytes[1] + r->L.gbytes[2]);
              if (rg.ty != ty || (b <= kCacheBytes) != fits) continue;
              if (fits && bytes + b > kCacheBytes) close();
              geom = rg;
              bytes += b;
              build_strips(r->p.nx, r->p.ny, slot, rg, g);
            }
            close();
          }
  // the resident set is marked clean only once its tables are on the device:
  // a failed rebuild leaves it dirty, so the next pump tries again
  if (all.empty()) {
    s->dirty = false;
    return NPLBM_OK;
  }
  // Waves: the groups that run side by side hold states that fit the 256 MB
  // Infinity Cache together, so the steps of a quantum read them from there;
  // the waves of a quantum run one after the other, each for all its steps
  // (20 FP32 requests of 64..432 a side, 1.0 M nodes and 330 MB: 70 us a
  // step against 85 with all groups side by side).  The groups beyond the
  // cache run side by side in a last wave, all domains of one kind in one
  // launch: in launches of their own each domain pays for a last round that
  // is partly empty (50 steps of six 1152 x 1200 N = 3 FP64 39.2 ms against
  // 48.1, of three with twelve FP32 of 200 a side 22.9 against 25.9).
  std::vector<int64_t> load;
  for (auto &gr : s->groups) {
    if (gr.bytes > kCacheBytes) continue;
    size_t w = 0;
    while (w < load.size() && load[w] + gr.bytes > kCacheBytes) ++w;
    if (w == load.size()) load.push_back(0);
    load[w] += gr.bytes;
    gr.wave = (int)w;
  }
  s->waves = (int)load.size();
  for (auto &gr : s->groups)
    if (gr.bytes > kCacheBytes) {
      gr.wave = (int)load.size();
      s->waves = gr.wave + 1;
    }
  if (all.size() > s->strips_cap) {
    if (s->strips_dev) (void)hipFree(s->strips_dev);
    s->strips_dev = nullptr;
    size_t cap = std::max(all.size() * 2, (size_t)1024);
    hipError_t e = hipMalloc(&s->strips_dev, cap * sizeof(StripDesc));
    if (e != hipSuccess) {
      s->strips_cap = 0;
      return hip_fail(e, "strip table allocation");
    }
    s->strips_cap = cap;
  }
  hipError_t e = hipMemcpyAsync(s->strips_dev, all.data(), all.size() * sizeof(StripDesc),
                                hipMemcpyHostToDevice, s->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(s->stream);  // `all` ends with this call
  if (e != hipSuccess) return hip_fail(e, "strip table upload");
  const int nside = s->groups.size() > 1 ? std::min((int)s->groups.size(), kSideStreams) : 0;
  while ((int)s->side.size() < nside) {
    hipStream_t st = nullptr;
    hipEvent_t ev = nullptr;
    e = hipStreamCreateWithFlags(&st, hipStreamNonBlocking);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
    if (e != hipSuccess) {
      if (st) (void)hipStreamDestroy(st);
      return hip_fail(e, "side stream creation");
    }
    s->side.push_back(st);
    s->join.push_back(ev);
  }
  if (nside && !s->fork) {
    e = hipEventCreateWithFlags(&s->fork, hipEventDisableTiming);
    if (e != hipSuccess) return hip_fail(e, "event creation");
  }
  s->dirty = false;
  return NPLBM_OK;
}

// Enqueue one quantum on the server's stream (eagerly or under capture).
// Groups touch disjoint domains and strip tables, so their chains of launches
// are independent: where a wave has more than one, each chain goes to a side
// stream forked from and joined back to the server's stream, and the groups
// run side by side (a small group does not leave the GPU half idle for a
// whole launch).
hipError_t enqueue_quantum(nplbm_server *s) {
  for (int w = 0; w < s->waves; ++w) {
    std::vector<const nplbm_server::Group *> gs;
    for (const auto &gr : s->groups)
      if (gr.wave == w) gs.push_back(&gr);
    const int nside = gs.size() > 1 ? std::min((int)gs.size(), kSideStreams) : 0;
    hipError_t e = hipSuccess;
    if (nside) {
      e = hipEventRecord(s->fork, s->stream);
      for (int j = 0; j < nside && e == hipSuccess; ++j)
        e = hipStreamWaitEvent(s->side[j], s->fork, 0);
    }
    for (int q = 0; q < s->quantum && e == hipSuccess; ++q)
      for (size_t gi = 0; gi < gs.size() && e == hipSuccess; ++gi) {
        const auto &gr = *gs[gi];
        StepArgs a;
        std::memset(&a, 0, sizeof a);
        a.strips = s->strips_dev + gr.off;
        a.doms = s->descs_dev;
        a.substep = q;
        e = launch_geom_step(gr.N, gr.precision, gr.scheme, gr.geom, a, (int)gr.count, nullptr,
                             nside ? s->side[gi % nside] : s->stream);
      }
    for (int j = 0; j < nside && e == hipSuccess; ++j) {
      e = hipEventRecord(s->join[j], s->side[j]);
      if (e == hipSuccess) e = hipStreamWaitEvent(s->stream, s->join[j], 0);
    }
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Capture the quantum of the present resident set as a graph.
int capture_quantum(nplbm_server *s) {
  hipGraph_t g = nullptr;
  hipError_t e = hipStreamBeginCapture(s->stream, hipStreamCaptureModeThreadLocal);
  if (e != hipSuccess) return hip_fail(e, "hipStreamBeginCapture");
  const hipError_t le = enqueue_quantum(s);
  e = hipStreamEndCapture(s->stream, &g);
  if (le != hipSuccess) {
    if (g) (void)hipGraphDestroy(g);
    return hip_fail(le, "step launch during capture");
  }
  if (e != hipSuccess) return hip_fail(e, "hipStreamEndCapture");
  e = hipGraphInstantiate(&s->graph, g, nullptr, nullptr, 0);
  (void)hipGraphDestroy(g);
  if (e != hipSuccess) {
    s->graph = nullptr;
    return hip_fail(e, "hipGraphInstantiate");
  }
  return NPLBM_OK;
}

// Publish the outcome of a request (under the mutex): done, with its
// latency recorded, or failed, with the error the admission or read-back
// raised.
void finish(nplbm_server *s, Req *r, int rc) {
  std::lock_guard<std::mutex> lk(s->mu);
  if (rc) {
    r->err = rc;
    r->msg = last_error();
    r->state = 3;
    return;
  }
  s->lat.push_back(r->t_done - r->t_submit);
  s->t_last = std::max(s->t_last, r->t_done);
  r->state = 2;
}

int retire(nplbm_server *s, Req *r) {
  const size_t n = (size_t)r->p.nx * r->p.ny;
  const int par = (int)(r->done_steps & 1);
  DomDesc D = r->desc;
  const size_t bytes = r->L.p + n * 8 - r->L.c;
  r->out.reset(new (std::nothrow) double[bytes / 8]);
  if (!r->out) {
    release(s, r);
    s->dirty = true;
    return fail(NPLBM_ENOMEM, "host memory for the results of %zu nodes", n);
  }
  auto dp = [&](size_t off) { return reinterpret_cast<double *>(r->base + off); };
  hipError_t e = launch_macro(s->descs_dev + r->slot, D, r->p.precision, par, dp(r->L.phi),
                              dp(r->L.rho), dp(r->L.C), dp(r->L.c), dp(r->L.u), dp(r->L.p),
                              r->L.q ? dp(r->L.q) : nullptr, s->stream);
  if (e == hipSuccess) e = copy_to_host(r->out.get(), dp(r->L.c), bytes, s->stream);
  if (e != hipSuccess) (void)hipStreamSynchronize(s->stream);
  release(s, r);
  s->dirty = true;
  if (e != hipSuccess) return hip_fail(e, "retire");
  r->t_done = now_s();
  s->completed += 1;
  return NPLBM_OK;
}

// Fail every resident request with the error of a quantum that broke off: what
// was enqueued of it has advanced some domains by an unknown part of the
// quantum, so none can be continued.  Waits for that work first.
void abandon(nplbm_server *s, int rc) {
  for (hipStream_t st : s->side) (void)hipStreamSynchronize(st);
  (void)hipStreamSynchronize(s->stream);
  for (size_t i = 0; i < s->slots.size(); ++i)
    if (Req *r = s->slots[i]) {
      release(s, r);
      finish(s, r, rc);
    }
  s->dirty = true;
}

}  // namespace

extern "C" {

int nplbm_server_create(size_t hbm_budget, int32_t max_slots, int32_t quantum, void *stream,
                        nplbm_server **out) {
  clear_error();
  if (!out) return fail(NPLBM_EINVAL, "out is NULL");
  *out = nullptr;
  if (max_slots < 1 || max_slots > 4096 || quantum < 1 || quantum > 100000 || hbm_budget == 0)
    return fail(NPLBM_EINVAL, "bad server limits");
  if (!stream) return fail(NPLBM_EINVAL, "the server needs a non-null stream (graph capture)");
  nplbm_server *s = new nplbm_server();
  s->budget = hbm_budget;
  s->max_slots = max_slots;
  s->quantum = quantum;
  s->stream = static_cast<hipStream_t>(stream);
  s->slots.assign(max_slots, nullptr);
  hipError_t e = hipMalloc(&s->descs_dev, sizeof(DomDesc) * (size_t)max_slots);
  if (e != hipSuccess) {
    forget_hip_error();
    delete s;
    return fail(NPLBM_ENOMEM, "descriptor table allocation: %s", hipGetErrorString(e));
  }
  *out = s;
  return NPLBM_OK;
}

int nplbm_submit(nplbm_server *s, const nplbm_params *p, const double *c, const double *u,
                 int64_t nsteps, uint64_t *ticket) {
  clear_error();
  if (!s || !p || !c || !ticket) return fail(NPLBM_EINVAL, "NULL argument");
  if (nsteps < 0) return fail(NPLBM_EINVAL, "nsteps < 0");
  if (is3d(p)) return fail(NPLBM_EINVAL, "the server takes 2-D domains (nz 0 or 1)");
  Req *r = new Req();
  int rc = derive(p, r->d);
  if (rc) {
    delete r;
    return rc;
  }
  const int N = p->N;
  r->sigma.assign(p->sigma, p->sigma + N * N);
  r->rho.assign(p->rho, p->rho + N);
  r->mu.assign(p->mu, p->mu + N);
  r->mob.assign(p->mobility, p->mobility + N - 1);
  r->tau.assign(p->tau_phi, p->tau_phi + N - 1);
  r->p = *p;
  r->p.sigma = r->sigma.data();
  r->p.rho = r->rho.data();
  r->p.mu = r->mu.data();
  r->p.mobility = r->mob.data();
  r->p.tau_phi = r->tau.data();
  r->L = plan_layout(&r->p);
  r->bytes = r->L.total;
  if (r->bytes > s->budget) {
    size_t b = r->bytes;
    delete r;
    return fail(NPLBM_ETOOBIG, "request needs %zu bytes, budget is %zu", b, s->budget);
  }
  const size_t n = (size_t)p->nx * p->ny;
  const size_t id = first_bad_sum(c, N, n);
  if (id < n) {
    delete r;
    return fail(NPLBM_EINVAL, "sum_k c_k != 1 at node %zu", id);
  }
  r->c.assign(c, c + (size_t)N * n);
  if (u) {
    r->u.assign(u, u + 2 * n);
    r->has_u = true;
  }
  r->nsteps = nsteps;
  r->t_submit = now_s();
  std::lock_guard<std::mutex> lk(s->mu);
  if (s->t_first < 0.0) s->t_first = r->t_submit;
  r->ticket = s->next_ticket++;
  s->reqs[r->ticket] = r;
  s->queue.push_back(r);
  *ticket = r->ticket;
  return NPLBM_OK;
}

int nplbm_server_pump(nplbm_server *s, int32_t *active_out) {
  clear_error();
  if (!s) return fail(NPLBM_EINVAL, "NULL server");
  const double t0 = now_s();
  // admission: first fit in arrival order
  std::vector<Req *> cand;
  {
    std::lock_guard<std::mutex> lk(s->mu);
    cand.assign(s->queue.begin(), s->queue.end());
  }
  int nres = 0;
  for (Req *r : s->slots) nres += r != nullptr;
  for (Req *r : cand) {
    if (nres >= s->max_slots) break;
    if (s->used + r->bytes > s->budget) continue;
    int rc = admit(s, r);
    {
      std::lock_guard<std::mutex> lk(s->mu);
      s->queue.erase(std::find(s->queue.begin(), s->queue.end(), r));
      if (!rc) r->state = 1;
    }
    if (!rc && r->nsteps == 0) rc = retire(s, r);
    else if (!rc) ++nres;
    if (rc || r->nsteps == 0) finish(s, r, rc);
  }
  // A resident set's first quantum is launched as it stands and captured as a
  // graph when it comes up again unchanged: sets change with every request
  // that finishes, and capturing and instantiating costs more (about 1.5 ms
  // for 50 steps of three groups) than one round of launches.
  const bool fresh = s->dirty;
  if (s->dirty) {
    int rc = rebuild(s);
    if (rc) return rc;
  }
  if (nres > 0 && s->waves == 0)
    return fail(NPLBM_ESTATE, "resident requests but nothing to launch");
  if (s->waves) {
    if (!fresh && !s->graph) {
      int rc = capture_quantum(s);
      if (rc) return rc;
    }
    // per-domain progress for this quantum
    double nodes = 0;
    hipError_t e = hipSuccess;
    for (int base = 0; base < s->max_slots && e == hipSuccess; base += kProgressSlots) {
      Progress pr{};
      pr.base = base;
      bool any = false;
      for (int j = 0; j < kProgressSlots; ++j) {
        Req *r = base + j < s->max_slots ? s->slots[base + j] : nullptr;
        pr.left[j] = -1;
        if (!r) continue;
        any = true;
        pr.left[j] = (int32_t)std::min<int64_t>(r->nsteps - r->done_steps, INT_MAX);
        if (r->done_steps & 1) pr.odd[j / 32] |= 1u << (j % 32);
        const int64_t adv = std::min<int64_t>(s->quantum, r->nsteps - r->done_steps);
        nodes += (double)adv * r->p.nx * r->p.ny;
      }
      if (any) e = launch_progress(s->descs_dev, pr, s->stream);
    }
    if (e != hipSuccess) return hip_fail(e, "progress upload");
    if (s->graph) {
      // a graph that was not launched left the state as it was: the next pump
      // tries again
      e = hipGraphLaunch(s->graph, s->stream);
      if (e != hipSuccess) return hip_fail(e, "hipGraphLaunch");
    } else {
      e = enqueue_quantum(s);
    }
    const char *what = e == hipSuccess ? "quantum" : "step launch";
    if (e == hipSuccess) e = hipStreamSynchronize(s->stream);
    if (e != hipSuccess) {
      const int rc = hip_fail(e, what);
      abandon(s, rc);
      return rc;
    }
    s->node_updates += nodes;
    for (int slot = 0; slot < s->max_slots; ++slot) {
      Req *r = s->slots[slot];
      if (!r) continue;
      r->done_steps += std::min<int64_t>(s->quantum, r->nsteps - r->done_steps);
      if (r->done_steps >= r->nsteps) finish(s, r, retire(s, r));
    }
  }
  if (active_out) {
    int a = 0;
    for (Req *r : s->slots) a += r != nullptr;
    *active_out = a;
  }
  s->busy += now_s() - t0;
  return NPLBM_OK;
}

int nplbm_poll(nplbm_server *s, uint64_t ticket, int32_t *state) {
  clear_error();
  if (!s || !state) return fail(NPLBM_EINVAL, "NULL argument");
  std::lock_guard<std::mutex> lk(s->mu);
  auto it = s->reqs.find(ticket);
  if (it == s->reqs.end()) return fail(NPLBM_ENOTFOUND, "unknown ticket");
  *state = it->second->state;
  return NPLBM_OK;
}

int nplbm_result(nplbm_server *s, uint64_t ticket, double *c, double *u, double *p,
                 double *admit_s, double *done_s) {
  clear_error();
  if (!s) return fail(NPLBM_EINVAL, "NULL server");
  Req *r = nullptr;
  {
    std::lock_guard<std::mutex> lk(s->mu);
    auto it = s->reqs.find(ticket);
    if (it == s->reqs.end()) return fail(NPLBM_ENOTFOUND, "unknown ticket");
    r = it->second;
    if (r->state == 3) {
      // a failed request is reaped here: its error is returned once
      s->reqs.erase(it);
      const int err = r->err ? r->err : NPLBM_EDEVICE;
      const std::string msg = r->msg;
      delete r;
      return fail(err, "request %llu failed: %s", (unsigned long long)ticket, msg.c_str());
    }
    if (r->state != 2) return fail(NPLBM_ESTATE, "request not finished (state %d)", r->state);
    s->reqs.erase(it);
  }
  const size_t n = (size_t)r->p.nx * r->p.ny;
  auto plane = [&](size_t off) { return r->out.get() + (off - r->L.c) / 8; };
  if (c) std::memcpy(c, plane(r->L.c), (size_t)r->p.N * n * 8);
  if (u) std::memcpy(u, plane(r->L.u), 2 * n * 8);
  if (p) std::memcpy(p, plane(r->L.p), n * 8);
  if (admit_s) *admit_s = r->t_admit - r->t_submit;
  if (done_s) *done_s = r->t_done - r->t_submit;
  delete r;
  return NPLBM_OK;
}

int nplbm_server_stats(nplbm_server *s, double *p50_s, double *p99_s, double *mlups,
                       double *node_updates, double *busy_s, int64_t *completed) {
  clear_error();
  if (!s) return fail(NPLBM_EINVAL, "NULL server");
  std::vector<double> lat;
  double span = 0.0;
  {
    std::lock_guard<std::mutex> lk(s->mu);
    lat = s->lat;
    span = s->t_first >= 0.0 ? s->t_last - s->t_first : 0.0;
  }
  // percentiles by linear interpolation between order statistics (rank
  // q (n - 1) of the sorted latencies)
  std::sort(lat.begin(), lat.end());
  auto pct = [&](double q) {
    if (lat.empty()) return 0.0;
    const double pos = q * (double)(lat.size() - 1);
    const size_t i = (size_t)pos;
    const double f = pos - (double)i;
    return i + 1 < lat.size() ? lat[i] + f * (lat[i + 1] - lat[i]) : lat[i];
  };
  if (p50_s) *p50_s = pct(0.50);
  if (p99_s) *p99_s = pct(0.99);
  if (mlups) *mlups = span > 0.0 ? s->node_updates / span / 1e6 : 0.0;
  if (node_updates) *node_updates = s->node_updates;
  if (busy_s) *busy_s = s->busy;
  if (completed) *completed = s->completed;
  return NPLBM_OK;
}

void nplbm_server_destroy(nplbm_server *s) {
  if (!s) return;
  for (hipStream_t st : s->side) (void)hipStreamSynchronize(st);
  (void)hipStreamSynchronize(s->stream);
  for (Req *r : s->slots)
    if (r) release(s, r);
  for (auto &kv : s->reqs) delete kv.second;
  if (s->graph) (void)hipGraphExecDestroy(s->graph);
  if (s->strips_dev) (void)hipFree(s->strips_dev);
  if (s->descs_dev) (void)hipFree(s->descs_dev);
  for (hipStream_t st : s->side) (void)hipStreamDestroy(st);
  for (hipEvent_t ev : s->join) (void)hipEventDestroy(ev);
  if (s->fork) (void)hipEventDestroy(s->fork);
  delete s;
}

}  // extern "C"
